"""Round limits reached inside the tail kernel, with energies asked for and
the workspace holding leftovers that pass for node counts and node numbers:
every limit is refused or accepted as by the CPU oracle, at whichever level it
is reached, and an accepted call's labels and energies are the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_00385_amd import ezsp, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ezsp.load()
    yield


def refill(ws):
    # the control block: negative counts; behind it a large node number
    words = ws[:ws.numel() // 4 * 4].view(torch.int32)
    words[:1 << 14].fill_(-0x40800000)
    words[1 << 14:].fill_(0x3F800000)


@pytest.mark.parametrize("d", [4, 13, 16])
@pytest.mark.parametrize("n", [1400, 2000])  # level 0 in the tail, or before
@pytest.mark.parametrize("lambdas", [[0.2], [3e-4, 6.0, 40.0],
                                     [6.0, 6.0, 40.0, 300.0]])
def test_limits_in_the_tail(n, d, lambdas):
    sc = scenes.random_cloud(n, d, seed=9)
    xyz, emb = torch.from_numpy(sc.xyz).cuda(), torch.from_numpy(sc.emb).cuda()
    codes = set()
    for cap in range(1, 30):
        part = ezsp.Partitioner(n, d, 10, lambdas, max_rounds=cap,
                                energy=True)
        refill(part.ws)
        try:
            ref = oracle.partition(sc.xyz, sc.emb, 10, lambdas, None, cap)
        except oracle.OracleError:
            with pytest.raises(ezsp.EzspError) as e:
                part(xyz, emb)
            codes.add(e.value.code)
            continue
        labels, nc, energy = part(xyz, emb)
        assert np.array_equal(labels.cpu().numpy(), ref[0])
        assert np.array_equal(nc, ref[1])
        np.testing.assert_allclose(energy, ref[2], rtol=1e-9)
        break
    assert codes == {ezsp.ERR_NOT_CONVERGED} and 2 < cap < 29
