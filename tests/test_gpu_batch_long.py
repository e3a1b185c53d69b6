"""Batches that take the kernel for long leaves, against the oracle: one workgroup a tile and leaf, which writes the histogram itself, and
several of few and of many epochs; leaves that end inside an epoch, of one row and of none beside them.

Statistics are small multiples of a power of two: every sum is exact and has to agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu

N_ROWS = 60_000
MANY = [31_300 + 97 * i for i in range(30)] + [1, 0, 512, 20_000]


@pytest.mark.parametrize("n_features,n_bins,wide,lengths", [
    (2000, 255, False, [N_ROWS]),
    (1999, 255, False, [N_ROWS, 40_001, 700, 0, 1]),
    (500, 256, False, [N_ROWS, 40_001, 20_000, 0, 1]),
    (70, 255, False, [N_ROWS]),
    (70, 255, False, [2_049, 2_600, 5_000, 9_999]),      # one epoch a workgroup
    (1999, 255, False, MANY),
    (2000, 63, False, MANY),
    (1990, 64, False, [N_ROWS + 5_000 * i for i in range(12)]),
    (200, 63, True, [N_ROWS, 40_001, 20_000, 0, 1]),
    (2000, 63, True, MANY),
])
def test_long_leaves_in_a_batch(n_features, n_bins, wide, lengths):
    print(f"long batch {n_features} x {n_bins} wide {wide} leaves {len(lengths)}", flush=True)
    rng = np.random.default_rng(n_features)
    bins = rng.integers(0, n_bins, size=(N_ROWS, n_features)).astype(np.uint8)
    grad = (rng.integers(-2, 3, size=N_ROWS) * 0.5).astype(np.float32)
    hess = (rng.integers(1, 4, size=N_ROWS) * 0.25).astype(np.float32)
    p = GpuProblem(bins, n_bins, grad, hess)
    lists = [np.sort(rng.choice(N_ROWS, size=n, replace=n > N_ROWS)).astype(np.int32) for n in lengths]
    offs = np.concatenate([[0], np.cumsum(lengths)])
    flat = torch.from_numpy(np.concatenate(lists)).to(p.dev)
    B.gbdt_set_wide_accumulation(wide)
    try:
        assert not B.gbdt_debug_batch_is_short(n_features, n_bins, offs, 256, 2 if wide else B.gbdt_debug_occupancy(n_bins, True))
        hists = B.gbdt_hist_build_batch(p.packed, N_ROWS, n_features, n_bins, flat, offs, p.grad, p.hess)
    finally:
        B.gbdt_set_wide_accumulation(False)
    features = np.unique(np.concatenate([[0, 1, 15, 16, 31, 32, 63, 64, n_features - 2, n_features - 1],
                                         rng.integers(0, n_features, size=60)]) % n_features)
    got = B.hist_to_numpy(hists)
    for k, idx in enumerate(lists):
        ref = p.oracle(idx, features=features)
        for name in ("grad", "hess", "count"):
            assert np.array_equal(got[k][features][name].astype(np.float64), ref[name].astype(np.float64)), (k, len(idx), name)
        assert (got[k]["count"].sum(axis=1) == len(idx)).all()
