"""Leaves on both sides of the lines between the build kernels, against the oracle: one workgroup a tile, which writes the histogram,
and several of one, two, three and more epochs each, every one of them a single unit; the last epoch full, short of a row, of one row.

Statistics are small multiples of a power of two: every sum is exact and has to agree bit for bit."""
import numpy as np
import pytest

from paper_1706_08359_amd import binding as B
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu

N_ROWS = 30_000


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n_features,n_bins", [(2000, 255), (1999, 256), (2000, 63), (1990, 16)])
def test_units_of_one_epoch_and_more(n_features, n_bins, wide):
    rng = np.random.default_rng(n_features)
    bins = rng.integers(0, n_bins, size=(N_ROWS, n_features)).astype(np.uint8)
    grad = (rng.integers(-2, 3, size=N_ROWS) * 0.5).astype(np.float32)
    hess = (rng.integers(1, 4, size=N_ROWS) * 0.25).astype(np.float32)
    p = GpuProblem(bins, n_bins, grad, hess)
    features = np.unique(np.concatenate([[0, 15, 16, 31, 32, 63, 64, n_features - 1], rng.integers(0, n_features, size=40)]))
    seen = set()
    B.gbdt_set_wide_accumulation(wide)
    try:
        for epochs in (1, 4, 5, 8, 16, 17, 24, 58):
            for n in (512 * epochs, 512 * epochs - 1, 512 * epochs - 511):
                print(f"units {n_features} x {n_bins} wide {wide} rows {n}", flush=True)
                for idx in (None, np.sort(rng.choice(N_ROWS, size=n, replace=False)).astype(np.int32)):
                    plan = B.gbdt_debug_leaf_plan(N_ROWS, n_features, n_bins, n, idx is not None)
                    if plan["one_unit_each"]:
                        seen.add(plan["short"])
                    got = B.hist_to_numpy(p.build(idx, n_leaf=n))[features]
                    ref = p.oracle(idx, n_leaf=n, features=features)
                    for k in ("grad", "hess", "count"):
                        assert np.array_equal(got[k].astype(np.float64), ref[k].astype(np.float64)), (n, plan, k)
    finally:
        B.gbdt_set_wide_accumulation(False)
    assert seen == ({1} if wide and n_bins > 64 else {0, 1})
