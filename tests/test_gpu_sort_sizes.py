"""The radix sort at the edges of its tiles and of its four size classes,
seen through what depends on it: component statistics (sizes and means are
wrong unless equal labels are together) for label widths of one to three
passes, and exact neighbours (each point must be in one bucket), both against
the CPU oracle, bit for bit; and workspaces that serve fewer points too."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_00385_amd import ezsp

pytestmark = pytest.mark.gpu
SIZES = [2, 1023, 1024, 1025, 4097, 65_536, 65_537, 524_288, 524_289,
         2_097_152, 2_097_153]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ezsp.load()
    yield


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("nc", [2, 3, 513, 1025, 70_000, 2_200_000])
def test_sorted_labels(n, nc):
    rng = np.random.default_rng(n + nc)
    lab = rng.integers(0, nc, n).astype(np.int32)
    lab[rng.random(n) < 0.3] = nc - 1
    emb = rng.standard_normal((n, 2)).astype(np.float32)
    size, mean, _ = ezsp.component_stats(torch.from_numpy(lab).cuda(), nc,
                                         torch.from_numpy(emb).cuda())
    rs, rm, _ = oracle.component_stats(lab, nc, emb)
    assert np.array_equal(size.cpu().numpy(), rs)
    assert np.array_equal(mean.cpu().numpy(), rm)


@pytest.mark.parametrize("n", SIZES[:-2] + [262_144, 262_145])
def test_neighbours(n):
    rng = np.random.default_rng(n)
    # a plane and a dense corner: voxels with one point and with many
    xyz = rng.random((n, 3), dtype=np.float32)
    xyz[:, 2] *= 0.01
    xyz[: n // 3] *= 0.02
    xyz = xyz[rng.permutation(n)]
    nbr, d2 = ezsp.knn(torch.from_numpy(xyz).cuda(), 5, want_d2=True)
    ref, rd2 = oracle.knn(xyz, 5, "brute" if n <= 3000 else "kdtree")
    assert np.array_equal(nbr.cpu().numpy(), ref)
    assert np.array_equal(d2.cpu().numpy(), rd2)


def test_workspaces_grow_with_n():
    lib = ezsp.load()
    sizes = sorted({m + e for m in SIZES + [1 << 25, 3_000_000]
                    for e in (-1, 0, 1, 4096)})
    for query in (lambda n: lib.ezsp_knn_workspace_size(n, 10),
                  lambda n: lib.ezsp_component_stats_workspace_size(n, 2, 8),
                  lambda n: lib.ezsp_purity_workspace_size(n, 9000, 500)):
        got = [query(n) for n in sizes if n > 0]
        assert got == sorted(got)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 1025, 9000, 32_768, 32_769])
@pytest.mark.parametrize("k", [3, 8, 9, 16, 17, 24, 25, 40])
def test_neighbours_of_both_walks(n, k):
    # few points to a wave and many: ties (a lattice), repeated points, lists
    # longer than the cloud, a last bucket partly filled, far-off points
    rng = np.random.default_rng(n + k)
    xyz = rng.integers(0, 12, (n, 3)).astype(np.float32)
    far = rng.random(n) < 0.05
    xyz[far] = (rng.random((int(far.sum()), 3)) * 1000).astype(np.float32)
    dense = rng.random(n) < 0.5
    xyz[dense] += (rng.random((int(dense.sum()), 3)) * 0.3).astype(np.float32)
    nbr, d2 = ezsp.knn(torch.from_numpy(xyz).cuda(), k, want_d2=True)
    ref, rd2 = oracle.knn(xyz, k, "brute" if n <= 3000 else "kdtree")
    assert np.array_equal(nbr.cpu().numpy(), ref)
    assert np.array_equal(d2.cpu().numpy(), rd2)
