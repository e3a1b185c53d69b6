"""Wide accumulation of finite values whose sum over an epoch of 512 rows is past the largest fp32 number: up to sixteen such
values in a cell are summed as any others.  A later epoch takes them back, or the sum becomes an infinity."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu


# 5 values of 3e38 are 2^130.1; 15 of them 2^131.7.  28 x 200 is a 32-byte tile (built whole or in halves), 10 x 200 a
# 16-byte one.
@pytest.mark.parametrize("n_features,n_bins", [(40, 16), (28, 64), (28, 200), (10, 200)])
@pytest.mark.parametrize("listed", [False, True])
@pytest.mark.parametrize("many", [5, 15])
def test_sums_past_fp32_in_an_epoch(n_features, n_bins, listed, many):
    n_rows = 1024                                   # two epochs of one workgroup
    print(f"huge sums {n_rows} x {n_features}, {n_bins} bins, {many} values, list {listed}", flush=True)
    big = np.float32(3e38)
    bins = np.zeros((n_rows, n_features), np.uint8)
    grad, hess = np.zeros(n_rows, np.float32), np.zeros(n_rows, np.float32)
    bins[:many], grad[:many], hess[:many] = 1, big, big                     # epoch 0
    bins[512:512 + many - 1], grad[512:512 + many - 1] = 1, -big            # epoch 1 leaves one of them
    p = GpuProblem(bins, n_bins, grad, hess)
    B.gbdt_set_wide_accumulation(True)
    try:
        got = B.hist_to_numpy(p.build(np.arange(n_rows, dtype=np.int32) if listed else None))
    finally:
        B.gbdt_set_wide_accumulation(False)
    assert (got["count"][:, 1] == 2 * many - 1).all() and (got["count"][:, 0] == n_rows - 2 * many + 1).all()
    # a value is rounded to a multiple of 2^-(k + kWideShift) = 2^79, 2^-49 of itself: nothing that fp32 shows
    assert (np.abs(got["grad"][:, 1].astype(np.float64) - big) <= 2.0 ** -23 * big).all()
    assert np.isposinf(got["hess"][:, 1]).all()
    assert (got["grad"][:, 0] == 0).all() and (got["hess"][:, 0] == 0).all()


@pytest.mark.parametrize("n_features,n_bins", [(40, 16), (28, 64), (28, 200), (10, 200)])
@pytest.mark.parametrize("listed", [False, True])
def test_small_values_beside_them(n_features, n_bins, listed):
    """Two values whose magnitudes sum to more than 2^128 (with the 0.2 % by which a sum is taken larger), and 510 multiples
    of the grid such an epoch has, 2^79, in another bin: exact, and within 5e-13 of the sum of magnitudes whatever they are."""
    n_rows = 512
    print(f"small values {n_rows} x {n_features}, {n_bins} bins, list {listed}", flush=True)
    rng = np.random.default_rng(n_bins)
    bins = np.zeros((n_rows, n_features), np.uint8)
    small = rng.permutation(np.arange(2, n_rows))
    bins[small] = 1 + (np.arange(510) % 3)[:, None].astype(np.uint8)
    grad, hess = np.full(n_rows, 2.0 ** 80, np.float32), np.full(n_rows, 2.0 ** 80, np.float32)
    grad[bins[:, 0] == 2] = -3 * 2.0 ** 79                                 # (an odd multiple, rounded by neither sign)
    hess[bins[:, 0] == 3] = rng.uniform(2.0 ** 78, 2.0 ** 90, 170)          # (not multiples)
    grad[:2] = hess[:2] = 1.7e38
    p = GpuProblem(bins, n_bins, grad, hess)
    B.gbdt_set_wide_accumulation(True)
    try:
        got = B.hist_to_numpy(p.build(np.arange(n_rows, dtype=np.int32) if listed else None))
    finally:
        B.gbdt_set_wide_accumulation(False)
    assert (got["grad"][:, 1] == np.float32(170 * 2.0 ** 80)).all() and (got["grad"][:, 2] == np.float32(-510 * 2.0 ** 79)).all()
    assert (got["hess"][:, 1] == np.float32(170 * 2.0 ** 80)).all() and (got["grad"][:, 3] == np.float32(170 * 2.0 ** 80)).all()
    third = hess[bins[:, 0] == 3].astype(np.float64).sum()
    assert (np.abs(got["hess"][:, 3] - third) <= 2.0 ** -24 * third + 5e-13 * 3.4e38).all()
    assert (np.abs(got["grad"][:, 0].astype(np.float64) - 2 * np.float64(np.float32(1.7e38))) <= 2.0 ** -23 * 3.4e38).all()
