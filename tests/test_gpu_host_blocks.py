"""Growers borrow a block of page-locked memory for a call.  A call whose search finds no scratch in the caller's workspace
enqueues nothing, so its block serves later calls as any other's."""
import threading

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
    before = B.gbdt_debug_host_blocks()
    assert before[0] >= 1
    B.gbdt_set_workspace(ws)
    try:
        for _ in range(12):
            with pytest.raises(B.GbdtError, match="-4"):
                grow(packed, 0, n_features, n_bins, empty, empty, most, 1.0, 1e-3)
    finally:
        B.gbdt_set_workspace(None)
    assert B.gbdt_debug_host_blocks() == before


def test_a_large_block_takes_the_place_of_a_small_one():
    """Four blocks are kept.  When calls of several threads have left four small ones, a call that needs a large one leaves that
    behind, so the next one like it allocates nothing."""
    B.gbdt_reset()
    n_rows, n_features, n_bins = 40_000, 600, 2
    bins = [torch.randint(0, 2, (n_rows, n_features), dtype=torch.uint8, device="cuda") for _ in range(6)]
    torch.cuda.synchronize()

    def pack(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                B.gbdt_bins_pack(bins[i], n_bins)                           # (buffers of its own: calls share nothing else)

    for _ in range(20):                                                     # (until four were borrowed at the same time)
        threads = [threading.Thread(target=pack, args=(i,)) for i in range(6)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        if B.gbdt_debug_host_blocks()[0] == 4:
            break
    kept, left, largest = B.gbdt_debug_host_blocks()
    assert left == 0 and kept <= 4
    wide = torch.randint(0, 2, (9000, 40_000), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        B.gbdt_bins_pack(wide, n_bins)
        assert B.gbdt_debug_host_blocks()[2] >= 4 * 40_000 and B.gbdt_debug_host_blocks()[0] <= 4
