"""Rows and windows at the edges of the contraction's chunks, against the CPU
oracle's ladder, labels bit for bit: hubs whose row fills an LDS window (and
gets slack), fills a chunk, or needs the global path; many short rows between
them, with few and with many merges a round, in the first and later rounds,
with and without the tail kernel."""
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


@pytest.fixture(params=["tail", "no_tail"])
def tail_mode(request, monkeypatch):
    if request.param == "no_tail":
        monkeypatch.setenv("EZSP_TAIL_NODES", "0")
    else:
        monkeypatch.delenv("EZSP_TAIL_NODES", raising=False)


@pytest.mark.parametrize("hub", [62, 63, 64, 65, 127, 500, 817, 818, 819, 1022,
                                 1023, 1024, 1025, 1500])
@pytest.mark.parametrize("noise", [0.02, 0.4])
def test_hub_rows(hub, noise, tail_mode):
    # ten hubs listed by `hub` points each, the points also in chains
    rng = np.random.default_rng(hub)
    hubs, d = 10, 8
    n = hubs * (hub + 1)
    star = np.repeat(np.arange(hubs), hub)
    nbr = np.full((n, 3), -1, np.int32)
    leaf = np.arange(hubs, n)
    nbr[leaf, 0] = star
    nbr[leaf[:-1], 1] = leaf[1:]
    far = rng.random(n) < 0.2
    nbr[far, 2] = rng.integers(0, n, int(far.sum()))
    emb = (rng.standard_normal((n // 6 + 1, d))[rng.integers(0, n // 6 + 1, n)]
           + noise * rng.standard_normal((n, d))).astype(np.float32)
    order = rng.permutation(n)  # old -> new
    table = np.full_like(nbr, -1)
    table[order] = np.where(nbr >= 0, order[nbr], -1)
    lambdas = [0.5, 4.0, 20.0]
    labels, nc, _ = ezsp.partition_from_knn(
        torch.from_numpy(table).cuda(), torch.from_numpy(emb).cuda(), lambdas)
    lo, hi, w = oracle.graph(table)
    ref, rnc, _, _ = oracle.partition_graph(emb, lo, hi, w, lambdas)
    assert np.array_equal(nc, rnc)
    assert np.array_equal(labels.cpu().numpy(), ref)


@pytest.mark.parametrize("sizes", [(128, 129, 4096, 4097), (5000, 5121, 6144),
                                   (70_000, 4097, 300)])
def test_giant_components(sizes, tail_mode):
    # components that absorb `sizes` points in one round: a block each, shared
    # by blocks, ragged last segments; then merges among and into them
    check_giants(sizes, 16)


@pytest.mark.parametrize("d", [8, 32, 13, 64])
def test_giant_components_by_width(d, tail_mode):
    # shared by blocks (8, 32), and by one block (any other width)
    check_giants((5000, 5121, 300), d)


def check_giants(sizes, d):
    rng = np.random.default_rng(sum(sizes))
    n = sum(sizes) + 3000
    nbr = np.full((n, 3), -1, np.int32)
    emb = (rng.standard_normal((n, d)) * 3).astype(np.float32)
    a = 0
    for m in sizes:
        nbr[a + 1:a + m, 0] = a  # a star around one point
        emb[a:a + m] = (rng.standard_normal(d) * 2 +
                        0.01 * rng.standard_normal((m, d))).astype(np.float32)
        a += m
    nbr[a:, 0] = rng.integers(0, n, n - a)
    nbr[:, 1] = np.where(rng.random(n) < 0.1, rng.integers(0, n, n), -1)
    order = rng.permutation(n)
    table = np.full_like(nbr, -1)
    table[order] = np.where(nbr >= 0, order[nbr], -1)
    e = np.empty_like(emb)
    e[order] = emb
    lambdas = [0.5, 8.0, 60.0]
    labels, nc, en = ezsp.partition_from_knn(
        torch.from_numpy(table).cuda(), torch.from_numpy(e).cuda(), lambdas,
        energy=True)
    lo, hi, w = oracle.graph(table)
    ref, rnc, ren, _ = oracle.partition_graph(e, lo, hi, w, lambdas)
    assert np.array_equal(nc, rnc)
    assert np.array_equal(labels.cpu().numpy(), ref)
    np.testing.assert_allclose(en, ren, rtol=1e-9)
