"""The last epoch of a leaf (512 rows), where rows and whole wavefronts (64 rows) may be missing: roots, lists and batches whose
lengths lie around both, for every bin capacity and tile width, with and without wide sums, with one workgroup a tile (the
histogram is written by it) and with several.

The gradients are multiples of 1/2 and the hessians of 1/4: every sum is exact and has to agree with the oracle bit for bit."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu

LENGTHS = [1, 63, 64, 65, 449, 511, 512, 513, 576, 1023, 1025, 2049]


def same(got_t, ref, what):
    got = B.hist_to_numpy(got_t)
    for k in ("grad", "hess", "count"):
        assert np.array_equal(got[k].astype(np.float64), ref[k].astype(np.float64)), (what, k)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n_features,n_bins", [(70, 63), (12, 64), (28, 255), (40, 255), (9, 256), (130, 16), (20, 9)])
def test_leaves_that_end_inside_an_epoch(n_features, n_bins, wide):
    print(f"last epoch {n_features} x {n_bins} wide {wide}", flush=True)
    n_rows = 40_000
    rng = np.random.default_rng(n_features + n_bins)
    bins = rng.integers(0, n_bins, size=(n_rows, n_features)).astype(np.uint8)
    grad = (rng.integers(-2, 3, size=n_rows) * 0.5).astype(np.float32)
    hess = (rng.integers(1, 4, size=n_rows) * 0.25).astype(np.float32)
    p = GpuProblem(bins, n_bins, grad, hess)
    B.gbdt_set_wide_accumulation(wide)
    try:
        for n in LENGTHS + [n_rows - 511, n_rows]:
            same(p.build(n_leaf=n), p.oracle(n_leaf=n), ("root", n))
        lists = [np.sort(rng.choice(n_rows, size=n, replace=False)).astype(np.int32) for n in LENGTHS + [30_001]]
        for idx in lists:
            same(p.build(idx), p.oracle(idx), ("list", len(idx)))
        offs = np.concatenate([[0], np.cumsum([len(i) for i in lists])])
        hists = B.gbdt_hist_build_batch(p.packed, n_rows, n_features, n_bins,
                                        torch.from_numpy(np.concatenate(lists)).to(p.dev), offs, p.grad, p.hess)
        for k, idx in enumerate(lists):
            same(hists[k], p.oracle(idx), ("batch", len(idx)))
    finally:
        B.gbdt_set_wide_accumulation(False)
