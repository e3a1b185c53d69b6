"""The reduction pass takes 1, 2, 4, 8 or 32 threads a cell after the number of partial blocks a leaf has, and writes whole
runs of a feature's bins with few; statistics of several lists are gathered by parts of the rows on large matrices.
Batches of leaves of few and many workgroups a tile, of every width of tile, odd and even bins, with empty leaves between,
against sums in 64 bits (narrow: 512 / (2^26 - 512) of the leaf's sum of magnitudes a bin, and fp32 roundings; wide: the exact sum
rounded to fp32, up to 1e-12 of the sum of magnitudes, which the second of a workgroup's two partial blocks decides)."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows,n_features,n_bins,sizes", [
    (40_000, 1100, 63, [3000, 0, 9000, 5000, 2100]), (40_000, 1100, 63, [39_000]), (20_000, 2100, 13, [9000, 2500, 0, 6000]),
    (20_000, 2100, 16, [19_999]), (30_000, 700, 255, [2100, 8000, 4100, 15_000]), (30_000, 555, 100, [29_000]),
    (60_000, 300, 64, [50_000, 0, 10_000]), (60_000, 75, 256, [0, 2049, 40_000]), (60_000, 20, 17, [60_000]),
    (120_000, 28, 255, [120_000]), (600_000, 130, 65, [20_000, 50_000, 0, 9_000, 2_500, 30_000])])
@pytest.mark.parametrize("wide", [False, True])
def test_reduction(n_rows, n_features, n_bins, sizes, wide):
    print(f"reduction {n_rows} x {n_features} x {n_bins} {sizes} wide={wide}", flush=True)
    rng = np.random.default_rng(n_features + n_bins)
    bins = rng.integers(0, n_bins, size=(n_rows, n_features), dtype=np.uint8)
    g = rng.normal(size=n_rows).astype(np.float32)
    h = rng.uniform(0.01, 1.0, size=n_rows).astype(np.float32)
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).cuda(), n_bins)
    gd, hd = torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    leaves = [np.sort(rng.choice(n_rows, size=s, replace=False)) for s in sizes]
    offs = np.concatenate([[0], np.cumsum(sizes)])
    idx = torch.from_numpy(np.concatenate(leaves).astype(np.int32)).cuda()
    B.gbdt_set_wide_accumulation(wide)
    try:
        got = B.gbdt_hist_build_batch(packed, n_rows, n_features, n_bins, idx, offs, gd, hd).cpu().numpy()
        lone = [B.gbdt_hist_build(packed, n_rows, n_features, n_bins, idx[a:b].contiguous(), int(b - a), gd, hd).cpu().numpy()
                for a, b in zip(offs, offs[1:])]
    finally:
        B.gbdt_set_wide_accumulation(False)
    for k, rows in enumerate(leaves):
        at = (bins[rows].astype(np.int64) + np.arange(n_features) * n_bins).reshape(-1)
        for w, stat in ((g, 0), (h, 1), (None, 2)):
            weights = np.ones(len(rows)) if w is None else w[rows].astype(np.float64)
            ref = np.bincount(at, np.repeat(weights, n_features), n_features * n_bins).reshape(n_features, n_bins)
            for name, hist in (("batch", got[k]), ("lone", lone[k])):
                if w is None:
                    assert np.array_equal(hist.view(np.uint32)[..., 2], ref), (name, k)
                else:
                    total = np.abs(weights).sum()
                    limit = 2.0 ** -23 * np.abs(ref) + 1e-12 * total if wide else 1e-5 * total
                    assert (np.abs(hist[..., stat] - ref) <= limit + 1e-30).all(), (name, k, stat)


def test_left_counts_with_and_without_empty_leaves():
    n, f, nb = 5000, 9, 40
    rng = np.random.default_rng(3)
    bins = rng.integers(0, nb, size=(n, f), dtype=np.uint8)
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).cuda(), nb)
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    for offs in ([0, 1200, 5000], [0, 0, 1200, 1200, 5000, 5000]):
        k = len(offs) - 1
        splits = torch.cat([B.split_record(i % f, 11, "cuda").reshape(1, 9) for i in range(k)])
        counts = torch.full((k,), -7, dtype=torch.int64, device="cuda")
        _, left = B.gbdt_partition_rows_batch(packed, n, f, nb, idx, offs, splits, n_left_out=counts)
        assert left.tolist() == [int((bins[a:b, i % f] <= 11).sum()) for i, (a, b) in enumerate(zip(offs, offs[1:]))]
