"""The edge loss's row layouts and ways of drawing the intra sample against
the CPU oracle: every lane count and chunking of D, rows of 4k, 2k and odd
slots, tables and embeddings off their vector alignment; a sample drawn from
listed keys, one whose threshold's bin overflows the list (equal words), one
that is a large part of the slots, and one that takes every intra pair.  Pair
counts and masks are bit-identical; the bars of the fp32 outputs are those of
test_gpu_widen."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_00385_amd import ezsp
from test_gpu_widen import AFF_ATOL, check_loss, dev, loss_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ezsp.load()
    yield


@pytest.mark.parametrize("d", [2, 4, 7, 16, 17, 20, 36, 64, 65, 68, 130, 132,
                               260, 300, 516, 700, 1024])
def test_row_layouts(d):
    emb, nbr, cls, word = loss_case(600, d, 9, 5, seed=d)
    for rho in (0.2, 1.0):
        check_loss(emb, nbr, cls, word, 4.0, rho)


@pytest.mark.parametrize("k", [2, 4, 5, 6, 8, 12, 17, 64])
@pytest.mark.parametrize("d", [12, 32])
def test_slots_and_alignment(k, d):
    emb, nbr, cls, word = loss_case(1001, d, k, 5, seed=k, messy=True)
    check_loss(emb, nbr, cls, word, 1.0, 0.3)
    ref, raff, rgrad, rsmp = oracle.edge_loss(emb, nbr, cls, word, 1.0, 0.3)
    e = torch.zeros(emb.size + 1, device="cuda")[1:].view(emb.shape)
    t = torch.zeros(nbr.size + 1, dtype=torch.int32, device="cuda")[1:] \
        .view(nbr.shape)
    e.copy_(dev(emb))
    t.copy_(dev(nbr))
    st, aff, grad, smp = ezsp.edge_loss(e, t, dev(cls),
                                        dev(word.view(np.int32)), 1.0, 0.3)
    assert st["n_intra_kept"] == ref["n_intra_kept"]
    assert np.array_equal(smp.cpu().numpy(), rsmp)
    np.testing.assert_allclose(aff.cpu().numpy(), raff, rtol=0, atol=AFF_ATOL)
    st2, aff2, grad2, smp2 = ezsp.edge_loss(
        e, t, dev(cls), dev(word.view(np.int32)), 1.0, 0.3,
        want_affinity=False, want_grad=False, want_sampled=False)
    assert aff2 is None and grad2 is None and smp2 is None
    assert st2 == st


@pytest.mark.parametrize("words", [1, 16, 1 << 32])
@pytest.mark.parametrize("rho", [0.05, 0.3, 0.7, 0.999])
def test_samples(words, rho):
    # 40,000 points: more intra pairs than the list holds, so equal words
    # take the general selection; rho = 0.7 keeps more than an eighth of the
    # slots, rho = 0.999 every intra pair
    emb, nbr, cls, word = loss_case(40_000, 8, 8, 12, seed=3,
                                    word_range=words)
    ref = check_loss(emb, nbr, cls, word, 1.0, rho)
    assert ref["n_intra"] > 16384
    assert (ref["n_intra_kept"] == ref["n_intra"]) == (rho == 0.999)


def test_non_finite_row():
    emb, nbr, cls, word = loss_case(700, 20, 6, 3, seed=1)
    for value in (np.nan, np.inf):
        bad = emb.copy()
        bad[699, 19] = value
        with pytest.raises(ezsp.EzspError) as e:
            ezsp.edge_loss(dev(bad), dev(nbr), dev(cls),
                           dev(word.view(np.int32)), 1.0, 0.3)
        assert e.value.code == ezsp.ERR_NONFINITE
