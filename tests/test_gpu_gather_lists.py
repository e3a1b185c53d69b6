"""Statistics gathered by parts of the lists, in more lists than one launch takes (300): batches of row lists, and levels of a
tree whose lists are segments of its row buffer.  All sums are exact (multiples of 1/4), so results are equal."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu

N, F, NB = 530_000, 100, 65                    # four tiles; grad and hess are past an XCD's L2


def _problem(seed):
    rng = np.random.default_rng(seed)
    bins = rng.integers(0, NB, size=(N, F), dtype=np.uint8)
    grad = rng.integers(-8, 9, size=N).astype(np.float32) / 4
    hess = rng.integers(1, 9, size=N).astype(np.float32) / 4
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).cuda(), NB)
    return rng, bins, grad, hess, packed, torch.from_numpy(grad).cuda(), torch.from_numpy(hess).cuda()


@pytest.mark.parametrize("n_leaves,start", [(299, 0), (300, 17), (301, 0), (640, 17)])
def test_batch_of_many_lists(n_leaves, start):
    print(f"gather of {n_leaves} lists from {start}", flush=True)
    rng, bins, grad, hess, packed, gd, hd = _problem(n_leaves)
    sizes = rng.integers(0, 2 * 300_000 // n_leaves, size=n_leaves)
    sizes[[3, n_leaves - 2]] = 0
    offs = start + np.concatenate([[0], np.cumsum(sizes)])
    rows = rng.integers(0, N, size=offs[-1]).astype(np.int32)
    got = B.gbdt_hist_build_batch(packed, N, F, NB, torch.from_numpy(rows).cuda(), offs, gd, hd).cpu().numpy()
    for k, (a, b) in enumerate(zip(offs, offs[1:])):
        at = (bins[rows[a:b]].astype(np.int64) + np.arange(F) * NB).reshape(-1)
        for stat, w in ((0, grad[rows[a:b]]), (1, hess[rows[a:b]])):
            ref = np.bincount(at, np.repeat(w.astype(np.float64), F), F * NB).reshape(F, NB)
            assert np.array_equal(got[k][..., stat], ref), (k, stat)
        assert np.array_equal(got[k].view(np.uint32)[..., 2], np.bincount(at, minlength=F * NB).reshape(F, NB)), k


def test_levels_of_many_segments():
    depth = 10
    _, bins, _, _, packed, gd, hd = _problem(1)
    nodes, order, _ = B.gbdt_grow_tree_depthwise(packed, N, F, NB, gd, hd, depth, 1.0, 1.0, 0.0)
    level = np.zeros(len(nodes), int)
    for k, nd in enumerate(nodes[1:], 1):
        level[k] = level[int(nd["parent"])] + 1
    assert (level == depth).sum() > 2 * 300    # (more than 300 smaller children)
    columns = torch.from_numpy(bins).cuda()
    rows = {0: torch.arange(N, dtype=torch.int32, device="cuda")}
    for k, nd in enumerate(nodes):
        idx = rows.pop(k)
        assert idx.numel() == nd["count"]
        if nd["left"] < 0:
            assert torch.equal(order[int(nd["row_begin"]):int(nd["row_begin"]) + int(nd["count"])], idx), k
        if k % 4 == 1 or nd["left"] < 0:       # (its split as the calls made one by one find it)
            hist = B.gbdt_hist_build(packed, N, F, NB, idx, idx.numel(), gd, hd)
            rec = B.split_to_dict(B.gbdt_best_split(hist, 1.0, 1.0))
            assert (rec["feature"], rec["bin"], rec["gain"]) == (nd["feature"], nd["bin"], nd["gain"]), k
        if nd["left"] >= 0:
            goes = columns[idx.long(), int(nd["feature"])] <= int(nd["bin"])
            rows[int(nd["left"])], rows[int(nd["right"])] = idx[goes], idx[~goes]


@pytest.mark.parametrize("n_rows,n_leaves", [(2 ** 20, 33), (2 ** 20, 31), (2 ** 20 - 1, 33)])
@pytest.mark.parametrize("n_features", [64, 70])
def test_wide_sums_gathered_by_parts(n_rows, n_leaves, n_features):
    """Two and three tiles in halves: gathered from 2^20 rows on if a leaf holds at most a 32nd of them."""
    print(f"gather by parts {n_rows} x {n_features}, {n_leaves} lists", flush=True)
    rng = np.random.default_rng(n_leaves)
    bins = rng.integers(0, 255, size=(n_rows, n_features), dtype=np.uint8)
    grad = rng.integers(-8, 9, size=n_rows).astype(np.float32) / 4
    hess = rng.integers(1, 9, size=n_rows).astype(np.float32) / 4
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).cuda(), 255)
    sizes = np.full(n_leaves, 2 ** 20 // 32 + (1 if n_leaves == 31 else 0))   # (just in, just out)
    sizes[[0, 2]] += [1000, -1000]
    offs = np.concatenate([[0], np.cumsum(sizes)])
    rows = rng.integers(0, n_rows, size=offs[-1]).astype(np.int32)            # (repeats are legal)
    B.gbdt_set_wide_accumulation(True)
    try:
        got = B.gbdt_hist_build_batch(packed, n_rows, n_features, 255, torch.from_numpy(rows).cuda(), offs,
                                      torch.from_numpy(grad).cuda(), torch.from_numpy(hess).cuda()).cpu().numpy()
    finally:
        B.gbdt_set_wide_accumulation(False)
    for k in (0, 1, 2, n_leaves - 1):
        mine = rows[offs[k]:offs[k + 1]]
        for f in (0, 31, 32, 63, n_features - 1):
            for stat, w in ((0, grad), (1, hess)):
                assert np.array_equal(got[k, f, :, stat], np.bincount(bins[mine, f], w[mine].astype(np.float64), 255)), (k, f, stat)
            assert np.array_equal(got[k, f].view(np.uint32)[:, 2], np.bincount(bins[mine, f], minlength=255)), (k, f)
