"""Purity by the counter table and by the sort against the CPU oracle, bit for
bit: products of components and classes on both sides of the table's limit,
class counts on both sides of the LDS histograms, blocks whose points hold
more distinct pairs than their hash takes in sixteen probes, one giant pair,
and a workspace queried for more components than the call has."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2512_00385_amd import ezsp
from test_gpu_widen import check_purity, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ezsp.load()
    yield


@pytest.mark.parametrize("n,nc,n_cls", [
    (2816, 1, 1), (2817, 700, 1), (5000, 1, 4096), (3000, 1024, 1024),
    (3000, 1025, 1024), (3000, 512, 2048), (3000, 500, 2049),
    (300_000, 3000, 801), (300_000, 2900, 801), (100_000, 90_000, 11)])
def test_counts(n, nc, n_cls):
    rng = np.random.default_rng(n + nc + n_cls)
    for kind in ("spread", "giant", "one"):
        label = rng.integers(0, nc, n).astype(np.int32)
        cls = rng.integers(0, n_cls, n).astype(np.int32)
        if kind != "spread":
            at = rng.random(n) < (0.6 if kind == "giant" else 2.0)
            label[at], cls[at] = nc // 2, n_cls // 2
        check_purity(label, nc, cls, n_cls)


def test_one_workspace_for_many_components():
    n, n_cls = 50_000, 40
    lib = ezsp.load()
    most = lib.ezsp_purity_workspace_size(n, n, n_cls)
    ws = torch.empty(most, dtype=torch.uint8, device="cuda")
    cls = torch.zeros(n, dtype=torch.int32, device="cuda")
    for nc in (1, 100, 9_999, 10_000, 10_001, n):
        assert lib.ezsp_purity_workspace_size(n, nc, n_cls) <= most
        label = torch.arange(n, dtype=torch.int32, device="cuda") % nc
        out = ezsp.PurityStats()
        rc = lib.ezsp_purity(label.data_ptr(), n, nc, cls.data_ptr(), n_cls,
                             None, None, ctypes.byref(out), ws.data_ptr(),
                             most, torch.cuda.current_stream().cuda_stream)
        assert rc == ezsp.OK and out.purity == 1.0 and out.n_present == 1


@pytest.mark.parametrize("n_cls", [1, 2, 4, 5, 8, 9, 16, 17, 33, 64, 65])
def test_narrow_rows(n_cls):
    # few lanes a component: more components than the grid takes in one step,
    # a last step partly filled, and empty components
    rng = np.random.default_rng(n_cls)
    n, nc = 300_000, min(280_001, 2_400_000 // n_cls)
    label = rng.integers(0, nc, n).astype(np.int32)
    cls = ((label * 7 + rng.integers(0, 3, n)) % n_cls).astype(np.int32)
    check_purity(label, nc, cls, n_cls)


@pytest.mark.parametrize("n", [2816 * 64 - 1, 2816 * 64, 1_000_003])
@pytest.mark.parametrize("nc,n_cls", [(1, 1), (1, 541), (10, 8), (300, 20),
                                      (500, 64), (511, 64), (513, 64),
                                      (16, 2048), (20, 2049)])
def test_small_tables_in_copies(n, nc, n_cls):
    rng = np.random.default_rng(n + nc)
    label = rng.integers(0, nc, n).astype(np.int32)
    cls = rng.integers(0, n_cls, n).astype(np.int32)
    check_purity(label, nc, cls, n_cls)
