"""The two ways of the edge loss's sample against the CPU oracle: pair by pair
where it is a small part of the pairs, through every row where it is a large
one, on both sides of the rule between them, with and without a gradient, for
tables of fewer slots than the rule looks at and of many tiles a block.  Counts
and masks are bit-identical; the bars of the fp32 outputs are those of
test_gpu_widen."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_00385_amd import ezsp
from test_gpu_widen import LOSS_RTOL, check_loss, dev, loss_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ezsp.load()
    yield


@pytest.mark.parametrize("n,k", [(9, 3), (150, 5), (1700, 8), (6000, 17)])
@pytest.mark.parametrize("d", [6, 12, 32, 68])
def test_shares(n, k, d):
    emb, nbr, cls, word = loss_case(n, d, k, 4, seed=n + d, messy=True)
    rng = np.random.default_rng(n)
    # distances of about sqrt(d): affinities of a tenth (an inter pair's loss,
    # -log(1 - a), is off by up to 2^-24 / a of itself in fp32)
    tau, seen = 0.4 * d ** 0.5, []
    for name, c in (("regions", cls), ("coin", rng.integers(0, 2, n)),
                    ("mixed", rng.integers(0, 13, n)),
                    ("one", np.zeros(n)), ("all", np.arange(n))):
        c = c.astype(np.int32)
        for rho in (0.0, 0.02, 0.1, 0.4, 0.8, 0.99):
            ref = check_loss(emb, nbr, c, word, tau, rho)
            st = ezsp.edge_loss(dev(emb), dev(nbr), dev(c),
                                dev(word.view(np.int32)), tau, rho,
                                want_affinity=False, want_grad=False,
                                want_sampled=False)[0]
            assert st["n_intra_kept"] == ref["n_intra_kept"], (name, rho)
            assert st["loss"] == pytest.approx(ref["loss"], rel=LOSS_RTOL,
                                               abs=1e-12), (name, rho)
            seen.append(ref["n_intra_kept"] / max(ref["n_edges"], 1))
    assert min(seen) == 0 and (n == 9 or max(seen) > 0.5)


@pytest.mark.parametrize("low", [0.01, 0.45])
def test_many_tiles(low):
    # 17M slots: five tiles a block and two bins of the histogram a thread.
    # `low` of the words lie below one bin, that bin's are the first tiles
    # (twice what a block stages before it flushes), and the sample ends
    # inside it
    n, k = 530_001, 32
    rng = np.random.default_rng(7)
    nbr = (np.arange(n)[:, None] + rng.integers(1, 2000, (n, k))) % n
    nbr = nbr.astype(np.int32)
    cls = rng.integers(0, 2, n).astype(np.int32)
    cls[:3000] = 0
    emb = rng.standard_normal((n, 4), dtype=np.float32)
    word = rng.integers(1 << 31, 1 << 32, (n, k), dtype=np.uint64)
    word = word.astype(np.uint32)
    small = rng.random((n, k)) < low
    word[small] &= 0x3fffffff
    first = word.reshape(-1)[:7 * 2048]
    first[:] = 0x40000000 + rng.integers(0, 1 << 17, first.size,
                                         dtype=np.uint32)
    owner = oracle.edge_loss(emb, nbr, cls, word, 1.0, 1.0)[3].astype(bool)
    intra = owner & (cls[:, None] == cls[nbr])
    below = int(np.count_nonzero(intra & (word < 0x40000000)))
    inside = int(np.count_nonzero(intra & (word < 0x80000000))) - below
    n_inter = int(owner.sum() - intra.sum())
    assert 8192 < inside < 16384  # fits the list, not a block's stage
    m = below + inside // 2
    ref = check_loss(emb, nbr, cls, word, 1.0, m / (m + n_inter))
    assert below < ref["n_intra_kept"] < below + inside
