"""gbdt_bins_pack and gbdt_bins_fuse at the edges of the blocks they work in (128 rows x 128 features, 16
features a load, rows at any alignment): the column copy byte for byte, the tiles through the root
histogram with exact sums, and a fused copy whose levels first show after the rows that are looked at first."""
import numpy as np
import pytest
import torch

from oracle import gbdt_oracle as orc
from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def exact_stats(rng, n):
    return ((rng.integers(-2, 3, size=n) * 0.5).astype(np.float32),
            (rng.integers(1, 4, size=n) * 0.25).astype(np.float32))


def same_root(packed, bins, nb, grad, hess):
    n, f = bins.shape
    got = B.hist_to_numpy(B.gbdt_hist_build(packed, n, f, nb, None, n, torch.from_numpy(grad).to(DEV),
                                            torch.from_numpy(hess).to(DEV)))
    ref = orc.hist_build(bins, nb, grad, hess)
    for k in ("grad", "hess", "count"):
        assert np.array_equal(got[k].astype(np.float64), ref[k].astype(np.float64)), k


@pytest.mark.parametrize("n_features", [1, 3, 15, 16, 17, 33, 127, 128, 129, 300])
@pytest.mark.parametrize("n_rows,n_bins", [(1, 64), (127, 255), (129, 16), (128, 63), (4200, 16), (4200, 256)])
def test_pack_block_edges(n_rows, n_features, n_bins):
    print(f"pack {n_rows} x {n_features}, {n_bins} bins", flush=True)
    rng = np.random.default_rng(n_rows * 7 + n_features)
    bins = rng.integers(0, n_bins, size=(n_rows, n_features)).astype(np.uint8)
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).to(DEV), n_bins, fuse=False)
    g = B.gbdt_debug_geometry(n_features, n_bins, n_rows)
    stride = (n_rows + 255) // 256 * 256
    base = (n_rows * g["row_bytes"] + 512 * 64 + 255) // 256 * 256
    cols = packed.cpu().numpy()[base:base + n_features * stride].reshape(n_features, stride)
    assert np.array_equal(cols[:, :n_rows], bins.T)
    same_root(packed, bins, n_bins, *exact_stats(rng, n_rows))


@pytest.mark.parametrize("n_features,late", [(40, 16), (1500, 5), (37, 64), (4096, 3), (4097, 4)])
def test_fuse_sees_levels_of_late_rows(n_features, late):
    """Only bins 0 and 1 at first; in the last rows some features reach `late` levels."""
    n_rows, nb = max(70_001, (1 << 25) // n_features + 1), 64
    assert 0 < B.gbdt_debug_fuse_sample_rows(n_rows, n_features) < n_rows - 3   # (a part is looked at first)
    print(f"fuse {n_features} features, late levels {late}", flush=True)
    rng = np.random.default_rng(n_features)
    bins = rng.integers(0, 2, size=(n_rows, n_features)).astype(np.uint8)
    bins[-3:, ::3] = late - 1
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).to(DEV), nb, fuse=False)
    n_cols, fused = B.gbdt_bins_fuse(torch.from_numpy(bins).to(DEV), nb, packed)
    levels = bins.max(axis=0).astype(np.uint32) + 1
    expect = B.gbdt_debug_fusion_plan(levels)[2]
    assert n_cols == (expect if expect <= 0.85 * n_features else 0)
    same_root(packed, bins, nb, *exact_stats(rng, n_rows))


@pytest.mark.parametrize("n_rows,looks_first", [(9000, False), ((1 << 25) // 50, False), ((1 << 25) // 50 + 1, True)])
def test_fuse_gives_up_on_full_features(n_rows, looks_first):
    """63 levels everywhere: no two features fit a column, and none are fused, whether the first rows already prove
    it or the whole matrix is read; levels that only late rows show are no reason to give up early."""
    assert (B.gbdt_debug_fuse_sample_rows(n_rows, 50) > 0) == looks_first
    rng = np.random.default_rng(1)
    bins = torch.from_numpy(rng.integers(0, 63, size=(n_rows, 50)).astype(np.uint8)).to(DEV)
    packed = B.gbdt_bins_pack(bins, 63, fuse=False)
    assert B.gbdt_bins_fuse(bins, 63, packed) == (0, None)
    bins %= 4
    bins[-1] = 62                              # (one row, the last: read only with the whole matrix)
    packed = B.gbdt_bins_pack(bins, 63, fuse=False)
    assert B.gbdt_bins_fuse(bins, 63, packed) == (0, None)
    bins[-1] = 3
    packed = B.gbdt_bins_pack(bins, 63, fuse=False)
    n_cols, fused = B.gbdt_bins_fuse(bins, 63, packed)
    assert n_cols == B.gbdt_debug_fusion_plan(np.full(50, 4, np.uint32))[2] and fused is not None
