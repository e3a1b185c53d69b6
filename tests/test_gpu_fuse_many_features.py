"""Levels found by gbdt_bins_fuse around the size of the page-locked block they are handed over in (512 records of 36
bytes, 4,608 levels), one call after the other so that larger and smaller matrices share the blocks."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_features", [1, 255, 4607, 4608, 4609, 9300, 40])
def test_levels_of_many_features(n_features):
    n_rows, nb = 300, 16
    print(f"fuse {n_rows} x {n_features}, {nb} bins", flush=True)
    rng = np.random.default_rng(n_features)
    levels = rng.integers(1, 9, size=n_features)
    bins = (rng.integers(0, 1 << 20, size=(n_rows, n_features)) % levels).astype(np.uint8)
    bins_d = torch.from_numpy(bins).cuda()
    packed = B.gbdt_bins_pack(bins_d, nb, fuse=False)
    n_cols, fused = B.gbdt_bins_fuse(bins_d, nb, packed)
    expect = B.gbdt_debug_fusion_plan(bins.max(axis=0).astype(np.uint32) + 1)[2]
    if n_features == 1:  # a lone column saves nothing
        assert fused is None
        return
    assert n_cols == expect and fused is not None
    ones = torch.ones(n_rows, device="cuda")
    got = B.hist_to_numpy(B.gbdt_hist_build(packed, n_rows, n_features, nb, None, n_rows, ones, ones))["count"]
    for f in (0, n_features // 2, n_features - 1):
        assert np.array_equal(got[f], np.bincount(bins[:, f], minlength=nb))
