"""gbdt_best_split_batch over the shapes where its walk over (feature, bin) pairs changes: 16, 32 and 64
lanes a row, one to four steps a row, groups that end inside a step, launches of few and of many
workgroups.  Against the oracle's scan of the same fp32 histograms: identical choice."""
import numpy as np
import pytest
import torch

from oracle import gbdt_oracle as orc
from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bins", [2, 15, 16, 17, 32, 33, 48, 64, 65, 128, 129, 192, 193, 255, 256])
@pytest.mark.parametrize("n_features,n_hists", [(1, 1), (17, 3), (33, 70), (300, 9)])
def test_split_batch_of_every_walk(n_features, n_hists, n_bins):
    print(f"split {n_hists} x {n_features} x {n_bins}", flush=True)
    rng = np.random.default_rng(n_bins * 1000 + n_features)
    shape = (n_hists, n_features, n_bins)
    h = np.zeros(shape, dtype=B.BIN_DTYPE)
    h["count"] = rng.integers(0, 60, size=shape)
    h["grad"] = (rng.normal(size=shape) * np.sqrt(h["count"])).astype(np.float32)
    h["hess"] = (rng.uniform(0.05, 0.25, size=shape) * h["count"]).astype(np.float32)
    t = torch.from_numpy(h.view(np.float32).reshape(shape + (3,)).copy()).to("cuda:0")
    got = B.splits_to_dicts(B.gbdt_best_split_batch(t, 1.0, 1e-3))
    for i in range(n_hists):
        ref = orc.best_split(orc.from_f32_hist(h["grad"][i], h["hess"][i], h["count"][i]), 1.0, 1e-3)
        assert (got[i]["feature"], got[i]["bin"]) == (ref["feature"], ref["bin"]), (i, got[i], ref)
        if ref["feature"] >= 0:
            assert got[i]["left_count"] == ref["left_count"]
            assert np.float32(ref["left_grad"]) == np.float32(got[i]["left_grad"])
