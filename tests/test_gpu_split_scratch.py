"""gbdt_best_split_batch of many histograms within a caller's workspace of gbdt_workspace_bytes, the one for a small matrix: one
workgroup a histogram hands nothing over and needs no scratch."""
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_features,n_bins,n_hists", [(8, 16, 512), (14, 2, 512), (12, 255, 2000), (20, 255, 512)])
def test_searches_within_a_callers_workspace(n_features, n_bins, n_hists):
    print(f"scratch of {n_hists} x {n_features} x {n_bins}", flush=True)
    ws = torch.empty(B.gbdt_workspace_bytes(100, n_features, n_bins), dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(n_hists)
    hists = torch.empty(n_hists, n_features, n_bins, 3, device="cuda")
    hists[..., 0] = torch.randint(-9, 10, hists.shape[:3], device="cuda", generator=g).float()
    hists[..., 1] = 1.0
    hists[..., 2] = torch.full(hists.shape[:3], 2, dtype=torch.int32, device="cuda").view(torch.float32)
    want = B.splits_to_dicts(B.gbdt_best_split_batch(hists, 1.0, 1e-3))
    B.gbdt_set_workspace(ws)
    try:
        got = B.splits_to_dicts(B.gbdt_best_split_batch(hists, 1.0, 1e-3))
    finally:
        B.gbdt_set_workspace(None)
    assert got == want and all(r["feature"] >= 0 for r in got)
