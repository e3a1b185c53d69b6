"""Tiles of 16 slots with 256 bins have cells of their own layout (rows of 16): the remainder tile, and with wide
accumulation the halves of main tiles.  Feature counts around the edges of tiles and halves, odd and even bins, root, list
(dense and sparse) and batch, several workgroups a tile and one, against sums in 64 bits."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


def _exact(bins, nb, g, h, rows):
    f = bins.shape[1]
    at = (bins[rows].astype(np.int64) + np.arange(f) * nb).reshape(-1)
    return [np.bincount(at, np.repeat(w, f), f * nb).reshape(f, nb) for w in
            (g[rows].astype(np.float64), h[rows].astype(np.float64), np.ones(len(rows)))]


def _check(got, ref, sum_g, sum_h, wide, what):
    """Narrow: 512 / (2^26 - 512) of the sum of magnitudes a bin, and half as much for fp32 roundings.  Wide: the exact
    sum rounded to fp32, up to 1e-12 of the sum of magnitudes."""
    got = got.cpu().numpy()
    assert np.array_equal(got.view(np.uint32)[..., 2], ref[2]), what
    for k, total in ((0, sum_g), (1, sum_h)):
        limit = 2.0 ** -23 * np.abs(ref[k]) + 1e-12 * total if wide else 1e-5 * total
        assert (np.abs(got[..., k] - ref[k]) <= limit + 1e-300).all(), (what, k)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n_rows,n_features,n_bins", [
    (513, 1, 65), (5000, 15, 256), (5000, 16, 255), (60_000, 17, 201), (60_000, 28, 255), (3000, 32, 256),
    (60_000, 33, 255), (60_000, 48, 130), (60_000, 49, 255), (400_000, 64, 256), (20_000, 75, 67), (150_000, 100, 255)])
def test_short_rows(n_rows, n_features, n_bins, wide):
    print(f"short rows {n_rows} x {n_features} x {n_bins} wide={wide}", flush=True)
    rng = np.random.default_rng(n_features * 7 + n_bins)
    bins = rng.integers(0, n_bins, size=(n_rows, n_features), dtype=np.uint8)
    bins[:, 0] = n_bins - 1                                    # a constant feature: one cell of every row
    g = rng.normal(size=n_rows).astype(np.float32)
    h = rng.uniform(0.01, 1.0, size=n_rows).astype(np.float32)
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).cuda(), n_bins)
    gd, hd = torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    lists = [np.sort(rng.choice(n_rows, size=max(1, int(n_rows * q)), replace=False)) for q in (0.6, 0.19, 0.02)]
    B.gbdt_set_wide_accumulation(wide)
    try:
        def sums(rows):
            return float(np.abs(g[rows]).sum(dtype=np.float64)), float(h[rows].sum(dtype=np.float64))
        everything = np.arange(n_rows)
        got = B.gbdt_hist_build(packed, n_rows, n_features, n_bins, None, n_rows, gd, hd)
        _check(got, _exact(bins, n_bins, g, h, everything), *sums(everything), wide, "root")
        for rows in lists:
            idx = torch.from_numpy(rows.astype(np.int32)).cuda()
            got = B.gbdt_hist_build(packed, n_rows, n_features, n_bins, idx, len(rows), gd, hd)
            _check(got, _exact(bins, n_bins, g, h, rows), *sums(rows), wide, len(rows))
        offs = np.concatenate([[0], np.cumsum([len(r) for r in lists])])
        idx = torch.from_numpy(np.concatenate(lists).astype(np.int32)).cuda()
        got = B.gbdt_hist_build_batch(packed, n_rows, n_features, n_bins, idx, offs, gd, hd)
        for k, rows in enumerate(lists):
            _check(got[k], _exact(bins, n_bins, g, h, rows), *sums(rows), wide, ("batch", k))
    finally:
        B.gbdt_set_wide_accumulation(False)
