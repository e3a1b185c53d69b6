"""Wide sums of 256 bins: from 384 * 1024 sparse rows on a batch, from half as many a list of a main tile and its remainder is
built from whole tiles, below in halves; from 2**23 rows of the matrix on a list of up to three tiles and a batch of two full ones.
Either way the exact sum rounded to fp32, up to 1e-12 of the leaf's sum of magnitudes."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu

MANY = 384 * 1024


def build_and_compare(bins, n_bins, sizes, rng):
    n_rows, n_features = bins.shape
    g = rng.normal(size=n_rows).astype(np.float32)
    h = rng.uniform(0.01, 1.0, size=n_rows).astype(np.float32)
    packed = B.gbdt_bins_pack(bins, n_bins)
    gd, hd = torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    offs = np.concatenate([[0], np.cumsum(sizes)])
    rows = rng.permutation(n_rows)[:offs[-1]]
    rows = np.concatenate([np.sort(rows[a:b]) for a, b in zip(offs, offs[1:])]).astype(np.int32)
    idx = torch.from_numpy(rows).cuda()
    listed = bins[idx.long()].cpu().numpy()
    B.gbdt_set_wide_accumulation(True)
    try:
        got = [B.gbdt_hist_build_batch(packed, n_rows, n_features, n_bins, idx, offs, gd, hd).cpu().numpy()]
        if len(sizes) == 1:
            got.append(B.gbdt_hist_build(packed, n_rows, n_features, n_bins, idx, sizes[0], gd, hd).cpu().numpy()[None])
    finally:
        B.gbdt_set_wide_accumulation(False)
    for k, (a, b) in enumerate(zip(offs, offs[1:])):
        mine = rows[a:b]
        at = (listed[a:b].astype(np.int64) + np.arange(n_features) * n_bins).reshape(-1)
        for stat, w in ((0, g), (1, h)):
            w = w[mine].astype(np.float64)
            ref = np.bincount(at, np.repeat(w, n_features), n_features * n_bins).reshape(n_features, n_bins)
            for one in got:
                assert (np.abs(one[k][..., stat] - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-12 * np.abs(w).sum() + 1e-300).all(), (k, stat)
        count = np.bincount(at, minlength=n_features * n_bins).reshape(n_features, n_bins)
        assert all(np.array_equal(one[k].view(np.uint32)[..., 2], count) for one in got), k


@pytest.mark.parametrize("n_features,n_bins", [(33, 256), (48, 201)])
@pytest.mark.parametrize("n_rows,sizes", [
    (5 * MANY // 2, [MANY // 2]), (5 * MANY // 2, [MANY // 2 - 1]), (5 * MANY // 2 - 1, [MANY // 2]),  # a fifth of the rows, or more
    (MANY + 4, [MANY // 13] * 12 + [0, MANY // 13]), (MANY, [MANY // 16] * 16), (MANY, [MANY // 16] * 15 + [MANY // 16 - 1]),
    (MANY, [MANY // 2, MANY // 2])])
def test_sparse_rows(n_features, n_bins, n_rows, sizes):
    print(f"wide sparse rows {n_rows} x {n_features} x {n_bins}, {len(sizes)} leaves of {sum(sizes)}", flush=True)
    rng = np.random.default_rng(n_rows + len(sizes))
    bins = rng.integers(0, n_bins, size=(n_rows, n_features), dtype=np.uint8)
    build_and_compare(torch.from_numpy(bins).cuda(), n_bins, sizes, rng)


@pytest.mark.parametrize("n_features", [64, 65, 96, 97])
@pytest.mark.parametrize("n_rows", [2 ** 23, 2 ** 23 - 1])
@pytest.mark.parametrize("sizes", [[MANY // 2], [MANY // 16] * 15 + [MANY // 16 + 1]])
def test_sparse_rows_of_large_matrices(n_features, n_rows, sizes):
    n_bins = 255
    print(f"wide sparse rows {n_rows} x {n_features} x {n_bins}, {len(sizes)} leaves of {sum(sizes)}", flush=True)
    torch.manual_seed(n_features)
    bins = torch.randint(0, n_bins, (n_rows, n_features), dtype=torch.uint8, device="cuda")
    build_and_compare(bins, n_bins, sizes, np.random.default_rng(n_rows + len(sizes)))
