"""Component statistics by label-sorted segments against the CPU oracle:
sizes, means and centroids bit-identical (exact integer sums) where a run of
equal labels ends inside a group of lanes, spans groups, spans blocks, or is
the whole input; for every row layout (16-byte vectors or single floats),
inputs of at most 512 points (another conversion) and more."""
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


def labels_of(kind, n, nc, rng):
    if kind == "one":
        return np.full(n, nc - 1, np.int32)
    if kind == "spread":
        return rng.integers(0, nc, n).astype(np.int32)
    lab = rng.integers(0, nc, n).astype(np.int32)  # one of half the points
    lab[rng.random(n) < 0.5] = nc // 2
    return lab


@pytest.mark.parametrize("n,nc", [(1, 1), (3, 2), (63, 5), (512, 9),
                                  (513, 300), (4097, 1), (40_001, 3001),
                                  (70_000, 65_537)])
@pytest.mark.parametrize("d", [1, 4, 5, 12, 16, 20, 33, 64])
def test_segments(n, nc, d):
    rng = np.random.default_rng(n * 64 + d)
    for kind in ("one", "spread", "giant"):
        lab = labels_of(kind, n, nc, rng)
        # values over many binades, so that some round at 2^-F
        emb = (rng.standard_normal((n, d)) *
               2.0 ** rng.integers(-30, 3, (n, d))).astype(np.float32)
        xyz = (rng.random((n, 3)) * 100 - 50).astype(np.float32)
        # rows at a 16-byte boundary and past one
        buf = torch.zeros(n * d + 1, device="cuda")
        for off in (0, 1):
            e = buf[off:off + n * d].view(n, d)
            e.copy_(torch.from_numpy(emb))
            for x in (xyz, None):
                got = ezsp.component_stats(
                    torch.from_numpy(lab).cuda(), nc, e,
                    None if x is None else torch.from_numpy(x).cuda())
                ref = oracle.component_stats(lab, nc, emb, x)
                for name, a, b in zip(("size", "mean", "centroid"), got, ref):
                    if a is not None:
                        assert np.array_equal(a.cpu().numpy(), b), \
                            (kind, off, x is None, name)


@pytest.mark.parametrize("n,d", [(1_100_003, 16), (1_100_003, 32),
                                 (1_100_003, 64), (3_000_001, 16)])
def test_long_segments(n, d):
    # up to 64 entries a group of lanes: several steps of a group, runs that
    # end within a step and runs carried across steps, groups and blocks
    rng = np.random.default_rng(n + d)
    lab = np.repeat(np.arange(n // 40, dtype=np.int32),
                    rng.integers(1, 201, n // 40))[:n]
    assert lab.size == n
    lab = lab[rng.permutation(n)]
    nc = int(lab.max()) + 1
    emb = rng.standard_normal((n, d), dtype=np.float32)
    xyz = rng.random((n, 3), dtype=np.float32) * 100
    got = ezsp.component_stats(*(torch.from_numpy(lab).cuda(), nc,
                                 torch.from_numpy(emb).cuda(),
                                 torch.from_numpy(xyz).cuda()))
    for a, b in zip(got, oracle.component_stats(lab, nc, emb, xyz)):
        assert np.array_equal(a.cpu().numpy(), b)


def test_segments_non_finite_and_range():
    lab = torch.zeros(1000, dtype=torch.int32, device="cuda")
    for value, code in ((float("nan"), ezsp.ERR_NONFINITE),
                        (float("-inf"), ezsp.ERR_NONFINITE),
                        (2.0 ** 40, ezsp.ERR_RANGE)):
        for where in ("emb", "xyz"):
            emb = torch.ones(1000, 6, device="cuda")
            xyz = torch.ones(1000, 3, device="cuda")
            (emb if where == "emb" else xyz)[999, 2] = value
            with pytest.raises(ezsp.EzspError) as e:
                ezsp.component_stats(lab, 1, emb, xyz)
            assert e.value.code == code
