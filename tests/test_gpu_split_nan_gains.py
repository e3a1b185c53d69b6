"""gbdt_best_split(_batch) with lambda = 0 and no least hessian, on histograms with bins of weight zero: a side without gradient
and hessian makes 0 / 0, and such a gain loses against every number wherever its threshold lies -- in the same lane as
the best one, in another lane, wavefront or workgroup -- and however many histograms are searched together."""
import numpy as np
import pytest
import torch

from oracle import gbdt_oracle as orc
from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


def _best(gains, admissible):
    """The first of the largest gains; the first admissible threshold where no gain is a number; None without any."""
    flat, ok = gains.reshape(-1), admissible.reshape(-1)
    number = ok & ~np.isnan(flat)
    if number.any():
        return int(np.flatnonzero(number)[np.argmax(flat[number])])
    return int(np.flatnonzero(ok)[0]) if ok.any() else None


# 2,000 x 255: 125 workgroups of a lone histogram; 20 x 255: several; the others one
@pytest.mark.parametrize("n_features,n_bins,n_hists", [(1, 3, 7), (9, 5, 40), (28, 16, 64), (28, 64, 33), (20, 255, 9), (130, 100, 70),
                                                       (2000, 255, 2)])
def test_gains_that_are_no_numbers_lose(n_features, n_bins, n_hists):
    print(f"nan gains {n_hists} x {n_features} x {n_bins}", flush=True)
    rng = np.random.default_rng(n_features + n_bins)
    shape = (n_hists, n_features, n_bins)
    h = np.zeros(shape, dtype=B.BIN_DTYPE)
    h["count"] = rng.integers(1, 40, size=shape)
    lead, tail = rng.integers(0, n_bins + 1, size=shape[:2]), rng.integers(0, n_bins + 1, size=shape[:2])
    lead[rng.random(shape[:2]) < 0.5] = min(2, n_bins - 1)                  # just before the first thresholds that are numbers
    at = np.arange(n_bins)
    live = (at >= lead[..., None]) & (at < n_bins - tail[..., None] // 3)
    h["grad"] = np.where(live, rng.integers(-9, 10, size=shape), 0)         # (whole numbers: ties, and sums that never round)
    h["hess"] = np.where(live, rng.integers(1, 5, size=shape), 0)
    h[-1]["grad"], h[-1]["hess"] = 0, 0                                     # nothing but 0 / 0
    t = torch.from_numpy(h.view(np.float32).reshape(shape + (3,)).copy()).cuda()
    together = B.splits_to_dicts(B.gbdt_best_split_batch(t, 0.0, 0.0))
    for i in range(n_hists):
        with np.errstate(all="ignore"):
            _, gains = orc.best_split(orc.from_f32_hist(h["grad"][i], h["hess"][i], h["count"][i]), 0.0, 0.0, return_gains=True)
        admissible = np.ones((n_features, n_bins), bool)
        admissible[:, -1] = False                                           # (every bin has samples, no hessian is negative)
        want = divmod(_best(gains, admissible), n_bins)
        alone = B.split_to_dict(B.gbdt_best_split(t[i].contiguous(), 0.0, 0.0))
        for got, how in ((together[i], "together"), (alone, "alone")):
            assert (got["feature"], got["bin"]) == want, (i, how, got, want)
            if np.isfinite(gains[want]):
                assert got["gain"] == np.float32(gains[want]), (i, how)
