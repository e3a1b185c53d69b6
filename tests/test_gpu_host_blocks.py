"""Growers borrow a block of page-locked memory for a call.  A call whose search finds no scratch in the caller's workspace
enqueues nothing, so its block serves later calls as any other's."""
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depthwise", [False, True])
def test_calls_without_scratch_leave_no_block_behind(depthwise):
    n_features, n_bins = 40, 255               # (several workgroups a search; an empty matrix is built without scratch)
    grow, most = (B.gbdt_grow_tree_depthwise, 3) if depthwise else (B.gbdt_grow_tree, 8)
    packed = torch.zeros(max(B.gbdt_bins_packed_bytes(0, n_features, n_bins), 256), dtype=torch.uint8, device="cuda")
    empty = torch.zeros(1, device="cuda")
    ws = torch.empty(256 * 1024, dtype=torch.uint8, device="cuda")
    nodes, _, _ = grow(packed, 0, n_features, n_bins, empty, empty, most, 1.0, 1e-3)
    assert len(nodes) == 1 and nodes[0]["feature"] == -1
    kept, left = B.gbdt_debug_host_blocks()
    assert kept >= 1
    B.gbdt_set_workspace(ws)
    try:
        for _ in range(12):
            with pytest.raises(B.GbdtError, match="-4"):
                grow(packed, 0, n_features, n_bins, empty, empty, most, 1.0, 1e-3)
    finally:
        B.gbdt_set_workspace(None)
    assert B.gbdt_debug_host_blocks() == (kept, left)
