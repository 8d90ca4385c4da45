"""Grid subsampling with both table entries against the CPU oracle, kept
indices bit-identical: cells and point indices that just fill 63 bits of one
word, that need one more (16-byte entries), and far more; every cell holding
several points, the smallest index early or late in the input."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_00385_amd import ezsp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ezsp.load()
    yield


@pytest.mark.parametrize("bits", [(0, 0, 0), (1, 1, 1), (16, 16, 16),
                                  (17, 16, 16), (16, 16, 17), (20, 20, 20)])
@pytest.mark.parametrize("n", [1, 2, 255, 20_000])
@pytest.mark.parametrize("order", ["random", "falling"])
def test_entries(bits, n, order):
    # 20,000 points take 15 index bits: 48 bits of cells fit, 49 do not
    rng = np.random.default_rng(sum(bits) + n)
    cell = np.stack([rng.integers(0, 1 << b, n) for b in bits], 1)
    cell[0] = 0  # the corners set the origin and the bits
    cell[-1] = [(1 << b) - 1 for b in bits]
    rep = rng.integers(0, n, n)
    rep[0], rep[-1] = 0, n - 1
    cell = cell[rep]
    if order == "falling":
        cell = cell[np.lexsort(cell.T[::-1])[::-1]]
    # steps of 1/4 stay inside a cell of 1; exact in fp32 to 2^20
    xyz = (cell + rng.integers(0, 4, (n, 3)) * 0.125).astype(np.float32)
    xyz[(cell == 0).all(1)] = 0.0
    ref = oracle.grid_subsample(xyz, 1.0)
    got = ezsp.grid_subsample(torch.from_numpy(xyz).cuda(), 1.0)
    assert np.array_equal(got.cpu().numpy(), ref)
