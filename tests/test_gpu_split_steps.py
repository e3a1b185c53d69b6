"""gbdt_best_split(_batch) where a wavefront's step of rows changes shape: 4 to 64 lanes a row, rows that end inside a
lane's bins or are shorter than them, a last step that is not full, one workgroup and several, one step a wavefront
and many; rows whose running sums round (the sum from left to right decides) next to rows whose sums do not;
constraints that leave denominators without a lower bound.  Against the oracle's scan: identical choice."""
import numpy as np
import pytest
import torch

from oracle import gbdt_oracle as orc
from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


def _hists(rng, shape, wide):
    h = np.zeros(shape, dtype=B.BIN_DTYPE)
    h["count"] = rng.integers(0, 60, size=shape)
    scale = np.ones(shape)
    if wide:
        rows = rng.random(shape[:2]) < 0.3
        scale[rows] = 2.0 ** rng.integers(-40, 40, size=shape)[rows]
    h["grad"] = (rng.normal(size=shape) * np.sqrt(h["count"]) * scale).astype(np.float32)
    h["hess"] = (rng.uniform(0.05, 0.25, size=shape) * h["count"] * scale).astype(np.float32)
    return h


@pytest.mark.parametrize("n_bins", [2, 3, 4, 5, 8, 16, 18, 31, 33, 62, 64, 66, 127, 130, 253, 256])
@pytest.mark.parametrize("n_features,n_hists,lam,mch,wide", [
    (1, 1, 1.0, 1e-3, False), (15, 2, 0.0, 0.0, False), (65, 1, 1.0, 1e-3, True), (67, 90, 0.5, 0.0, True),
    (259, 40, 1.0, 1e-3, False)])
def test_steps_against_oracle(n_features, n_hists, lam, mch, wide, n_bins):
    print(f"split steps {n_hists} x {n_features} x {n_bins}", flush=True)
    rng = np.random.default_rng(n_bins * 7919 + n_features)
    shape = (n_hists, n_features, n_bins)
    h = _hists(rng, shape, wide)
    if n_features > 2:  # a tie across steps: the smaller feature wins
        h[0, -1] = h[0, 0]
    t = torch.from_numpy(h.view(np.float32).reshape(shape + (3,)).copy()).to("cuda:0")
    got = B.splits_to_dicts(B.gbdt_best_split_batch(t, lam, mch))
    for i in range(n_hists):
        with np.errstate(all="ignore"):
            ref = orc.best_split(orc.from_f32_hist(h["grad"][i], h["hess"][i], h["count"][i]), lam, mch)
        assert (got[i]["feature"], got[i]["bin"]) == (ref["feature"], ref["bin"]), (i, got[i], ref)
        if ref["feature"] >= 0:
            assert got[i]["left_count"] == ref["left_count"] and got[i]["right_count"] == ref["right_count"]
            assert np.float32(ref["left_grad"]) == np.float32(got[i]["left_grad"])
            assert np.float32(ref["right_hess"]) == np.float32(got[i]["right_hess"])


@pytest.mark.parametrize("n_bins", [3, 17, 65, 200])
def test_siblings_formed_in_the_search(n_bins):
    """Depth-wise growth forms siblings in the search and keeps all but the last level's; the tree is that of the
    calls made one by one."""
    n, f, depth = 6000, 21, 4
    rng = np.random.default_rng(n_bins)
    bins = rng.integers(0, n_bins, size=(n, f), dtype=np.uint8)
    grad = torch.from_numpy((rng.integers(0, 2, size=n) - 0.5 + 0.25 * (bins[:, 3] > n_bins // 2)).astype(np.float32)).cuda()
    hess = torch.full((n,), 0.25, device="cuda")
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).cuda(), n_bins)
    nodes, _, _ = B.gbdt_grow_tree_depthwise(packed, n, f, n_bins, grad, hess, depth, 1.0, 1e-3, 0.0)
    rows = {0: torch.arange(n, dtype=torch.int32, device="cuda")}
    assert len(nodes) > 15
    for k, nd in enumerate(nodes):
        idx = rows.pop(k)
        assert idx.numel() == nd["count"]
        hist = B.gbdt_hist_build(packed, n, f, n_bins, idx, idx.numel(), grad, hess)
        rec = B.split_to_dict(B.gbdt_best_split(hist, 1.0, 1e-3))   # (all sums are exact: multiples of 1/4)
        assert (rec["feature"], rec["bin"]) == (nd["feature"], nd["bin"]) and rec["gain"] == nd["gain"], k
        if nd["left"] >= 0:
            goes = torch.from_numpy(bins[:, nd["feature"]]).cuda()[idx.long()] <= int(nd["bin"])
            rows[int(nd["left"])], rows[int(nd["right"])] = idx[goes], idx[~goes]


@pytest.mark.parametrize("spread", [30, 60])
@pytest.mark.parametrize("n_bins", [5, 9, 16, 31, 63, 64, 100, 128, 200, 256])
def test_sums_that_round_are_the_ones_from_left_to_right(n_bins, spread):
    """Every feature holds the same bins, in an order of its own on either side of the one good threshold: gains differ by the
    rounding of the sums alone, and which is largest says whether those are the oracle's to the last bit."""
    n_features, n_hists, lam = 75, 24, 2.0 ** -10      # (lam: the same in fp32)
    print(f"rounding sums {n_hists} x {n_features} x {n_bins}, 2^+-{spread}", flush=True)
    rng = np.random.default_rng(n_bins + spread)
    h = np.zeros((n_hists, n_features, n_bins), dtype=B.BIN_DTYPE)
    t = n_bins // 2
    for i in range(n_hists):
        scale = 2.0 ** rng.integers(-spread, 1, size=n_bins) * (1 + i)
        grad = (rng.uniform(0.5, 1, size=n_bins) * np.where(np.arange(n_bins) < t, 1, -1) * scale).astype(np.float32)
        hess = (rng.uniform(0.5, 1, size=n_bins) * scale ** 0.5).astype(np.float32)
        for f in range(n_features):
            order = np.concatenate([rng.permutation(t), t + rng.permutation(n_bins - t)])
            h["grad"][i, f], h["hess"][i, f] = grad[order], hess[order]
    h["count"] = 3
    d = torch.from_numpy(h.view(np.float32).reshape(h.shape + (3,)).copy()).to("cuda:0")
    got = B.splits_to_dicts(B.gbdt_best_split_batch(d, lam, 0.0))
    filtered = B.splits_to_dicts(B.gbdt_best_split_batch(d, lam, 1e-30))
    for i in range(n_hists):
        ref = orc.best_split(orc.from_f32_hist(h["grad"][i], h["hess"][i], h["count"][i]), lam, 0.0)
        for one in (got[i], filtered[i]):
            assert (one["feature"], one["bin"]) == (ref["feature"], ref["bin"]), (i, one, ref)
