"""CPU-only checks of the built C-ABI library: it loads, exports every symbol the
header declares, rejects bad arguments before touching a GPU, and its host-side
launch planning (tiles, slots, chunks, workspace) is self-consistent."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_1706_08359_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    lib = B.load()
    header = open(os.path.join(ROOT, "include", "gbdt_hist.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(gbdt_[a-z_]+)\s*\(", header))
    assert declared, "no declarations found"
    assert declared == set(B.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


def test_strerror():
    assert B.gbdt_strerror(0) == "ok"
    assert "invalid" in B.gbdt_strerror(-1)
    assert "unknown" in B.gbdt_strerror(-99)


def test_argument_errors_are_rejected_before_any_gpu_work():
    lib = B.load()
    EINVAL, EUNSUP = -1, -2
    assert lib.gbdt_bins_packed_bytes(10, 0, 64) == 0
    assert lib.gbdt_bins_packed_bytes(10, 5, 1) == 0
    assert lib.gbdt_bins_packed_bytes(10, 5, 257) == 0
    assert lib.gbdt_bins_packed_bytes(-1, 5, 64) == 0
    assert lib.gbdt_workspace_bytes(10, 5, 300) == 0
    one = ctypes.c_void_p(256)    # never dereferenced: all calls below fail validation first
    assert lib.gbdt_bins_pack(None, 10, 5, 64, one, None) == EINVAL
    assert lib.gbdt_bins_pack(one, 10, 5, 64, None, None) == EINVAL
    assert lib.gbdt_bins_pack(one, 10, 5, 64, ctypes.c_void_p(260), None) == EINVAL   # misaligned
    assert lib.gbdt_bins_pack(one, 10, 5, 1, one, None) == EINVAL
    assert lib.gbdt_bins_pack(one, 1 << 31, 5, 64, one, None) == EUNSUP
    assert lib.gbdt_hist_build(one, 10, 5, 64, None, 5, one, one, None, None) == EINVAL
    assert lib.gbdt_hist_build(None, 10, 5, 64, None, 5, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build(one, 10, 5, 64, None, 5, None, one, one, None) == EINVAL
    assert lib.gbdt_hist_build(one, 10, 5, 64, None, 5, one, None, one, None) == EINVAL
    assert lib.gbdt_hist_build(one, 10, 5, 64, None, 11, one, one, one, None) == EINVAL   # root leaf > n_rows
    assert lib.gbdt_hist_build(one, 10, 5, 64, None, -1, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build(one, 10, 5, 0, None, 5, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build(one, 10, 5, 257, None, 5, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build(one, 10, 0, 64, None, 5, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build(one, 1 << 31, 5, 64, None, 5, one, one, one, None) == EUNSUP
    assert lib.gbdt_hist_subtract(None, one, one, 5, 64, None) == EINVAL
    assert lib.gbdt_hist_subtract(one, None, one, 5, 64, None) == EINVAL
    assert lib.gbdt_hist_subtract(one, one, None, 5, 64, None) == EINVAL
    assert lib.gbdt_hist_subtract(one, one, one, 5, 1, None) == EINVAL
    assert lib.gbdt_best_split(None, 1.0, 0.0, one, 5, 64, None) == EINVAL
    assert lib.gbdt_best_split(one, 1.0, 0.0, None, 5, 64, None) == EINVAL
    assert lib.gbdt_best_split(one, -1.0, 0.0, one, 5, 64, None) == EINVAL
    assert lib.gbdt_best_split(one, float("nan"), 0.0, one, 5, 64, None) == EINVAL
    assert lib.gbdt_best_split(one, 1.0, 0.0, one, 0, 64, None) == EINVAL
    # batched build: the offsets are a HOST array, validated before anything else happens
    offs = lambda *v: (ctypes.c_int64 * len(v))(*v)
    B.load()
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, one, offs(0, 3, 7), -1, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, one, offs(0, 3, 7), 0, one, one, one, None) == 0
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, one, None, 2, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, one, offs(0, 3, 7), 2, one, one, None, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, one, offs(0, 7, 3), 2, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, one, offs(-1, 3, 7), 2, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, None, offs(0, 3, 7), 2, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(None, 10, 5, 64, one, offs(0, 3, 7), 2, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 10, 5, 64, one, offs(0, 3, 7), 2, None, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 10, 5, 1, one, offs(0, 3, 7), 2, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 0, 5, 64, one, offs(0, 3, 7), 2, one, one, one, None) == EINVAL
    assert lib.gbdt_hist_build_batch(one, 1 << 31, 5, 64, one, offs(0, 3, 7), 2, one, one, one, None) == EUNSUP
    assert lib.gbdt_hist_build_batch_workspace_bytes(5, 1, 4) == 0
    assert lib.gbdt_hist_build_batch_workspace_bytes(5, 64, -1) == 0
    assert lib.gbdt_best_split_batch(one, -1, 1.0, 0.0, one, 5, 64, None) == EINVAL
    assert lib.gbdt_best_split_batch(one, 0, 1.0, 0.0, one, 5, 64, None) == 0
    assert lib.gbdt_best_split_batch(None, 2, 1.0, 0.0, one, 5, 64, None) == EINVAL
    assert lib.gbdt_best_split_batch(one, 2, 1.0, 0.0, None, 5, 64, None) == EINVAL
    assert lib.gbdt_best_split_batch(one, 2, -1.0, 0.0, one, 5, 64, None) == EINVAL
    assert lib.gbdt_partition_rows(None, 10, 5, 64, None, 5, one, one, one, None) == EINVAL
    assert lib.gbdt_partition_rows(one, 10, 5, 64, None, 5, None, one, one, None) == EINVAL
    assert lib.gbdt_partition_rows(one, 10, 5, 64, None, 5, one, None, one, None) == EINVAL
    assert lib.gbdt_partition_rows(one, 10, 5, 64, None, 11, one, one, one, None) == EINVAL
    assert lib.gbdt_partition_rows(one, 10, 5, 64, None, -1, one, one, one, None) == EINVAL
    assert lib.gbdt_partition_rows(one, 1 << 31, 5, 64, None, 5, one, one, one, None) == EUNSUP
    assert lib.gbdt_set_workspace(one, 0) == EINVAL
    assert lib.gbdt_set_workspace(None, 16) == EINVAL
    assert lib.gbdt_set_workspace(ctypes.c_void_p(100), 1024) == EINVAL               # misaligned
    assert lib.gbdt_set_workspace(None, 0) == 0


SHAPES = [(1, 2), (3, 16), (4, 17), (27, 63), (28, 64), (28, 255), (33, 64), (64, 64), (65, 65),
          (100, 256), (137, 255), (129, 16), (130, 16), (255, 16), (257, 16), (700, 16),
          (2000, 63), (2001, 63), (2047, 64), (968, 255)]


@pytest.mark.parametrize("n_features,n_bins", SHAPES)
def test_tile_plan_is_a_bijection_onto_slots(n_features, n_bins):
    g = B.gbdt_debug_geometry(n_features, n_bins, 1000)
    assert g["cap"] >= n_bins and g["cap"] in (16, 64, 256)
    assert g["nib"] == (1 if n_bins <= 16 else 0)
    assert g["wm"] == (32 if g["cap"] == 256 else 64) and g["wr"] in (0, 16, 32) and g["wr"] < g["wm"]
    assert g["row_bytes"] == g["n_main"] * g["wm"] + g["wr"]
    per_byte = 2 if g["nib"] else 1
    assert g["feat_bytes"] == (n_features + per_byte - 1) // per_byte
    assert g["feat_bytes"] <= g["row_bytes"] < g["feat_bytes"] + g["wm"] // 2 + 16
    # tiles, the slack the build kernels may read past them, then one byte per value column by column
    tiles = (12345 * g["row_bytes"] + 512 * 64 + 255) // 256 * 256
    assert B.gbdt_bins_packed_bytes(12345, n_features, n_bins) == tiles + n_features * ((12345 + 255) // 256 * 256)
    seen = set()
    for f in range(n_features):
        t, s = B.gbdt_debug_locate(n_features, n_bins, f)
        w = g["wm"] if t < g["n_main"] else g["wr"]
        assert 0 <= t < g["n_main"] + (1 if g["wr"] else 0) and w > 0
        assert 0 <= s < w * per_byte
        assert (t, s) not in seen
        seen.add((t, s))
    # the main tile's histogram (8-byte cells, 32 slots per page row) must fit the LDS
    # the kernel declares, and the CU
    pages = (g["wm"] * per_byte + 31) // 32
    assert pages * g["cap"] * 32 * 8 <= g["lds_bytes"] <= 160 * 1024


@pytest.mark.parametrize("n_features,n_bins", [(28, 64), (2000, 63), (28, 255), (137, 255), (700, 16), (5, 2)])
@pytest.mark.parametrize("n_leaf", [1, 63, 64, 65, 511, 512, 513, 4000, 100_003, 266_000, 10_500_000])
def test_workgroups_per_tile(n_features, n_bins, n_leaf):
    g = B.gbdt_debug_geometry(n_features, n_bins, n_leaf)
    per_byte = 2 if g["nib"] else 1
    n_epochs = (n_leaf + 511) // 512
    n_tiles = g["n_main"] + (1 if g["wr"] else 0)
    wgs, k = g["wgs"], g["unit_epochs"]
    # the grid fits the machine once; every workgroup's first unit exists
    assert wgs >= 1 and k >= 1 and wgs * n_tiles <= max(256 * 4, n_tiles)
    n_units = (n_epochs + k - 1) // k
    assert wgs <= max(n_units, 1)
    # units beyond a workgroup's first come from the tile's counter; the two epochs of
    # look-ahead across a unit's end need units of at least 3 epochs then
    assert n_units <= wgs or k >= 3
    words = 0
    for w, tiles in ((g["wm"], g["n_main"]), (g["wr"], 1 if g["wr"] else 0)):
        pages = (w * per_byte + 31) // 32
        words += tiles * wgs * 3 * g["cap"] * 32 * pages
    assert words == g["partial_words"]
    assert B.gbdt_workspace_bytes(n_leaf, n_features, n_bins) >= 4 * (g["partial_words"] + n_tiles)
    assert n_tiles * wgs < 2 ** 31


@pytest.mark.parametrize("n_features,n_bins,wg_per_cu", [(28, 255, 2), (2000, 63, 3), (700, 16, 4), (137, 255, 2), (40, 64, 3)])
def test_batched_launch_plan_covers_every_leaf_exactly(n_features, n_bins, wg_per_cu):
    """Host planning of gbdt_hist_build_batch and the block -> (leaf, tile, workgroup) mapping
    the kernel uses: every (leaf, tile, workgroup) is hit by exactly one block, empty leaves get
    none, and a leaf's workgroups (unit c, c + wgs, ...) cover each of its epochs exactly once."""
    rng = np.random.default_rng(n_features + n_bins)
    geo = B.gbdt_debug_geometry(n_features, n_bins, 1)
    n_tiles = geo["n_main"] + (1 if geo["wr"] else 0)
    for trial in range(12):
        n_leaves = int(rng.integers(1, 129))
        kind = trial % 4
        if kind == 0:
            sizes = rng.integers(0, 3000, size=n_leaves)
        elif kind == 1:
            sizes = rng.integers(0, 2, size=n_leaves) * rng.integers(1, 200_000, size=n_leaves)
        elif kind == 2:
            sizes = np.full(n_leaves, 1)
            sizes[0] = 3_000_000
        else:
            sizes = (2_000_000 * rng.dirichlet(np.ones(n_leaves))).astype(np.int64)
        offs = np.concatenate([[5], 5 + np.cumsum(sizes)])
        wgs, ue, blocks = B.gbdt_debug_batch_plan(n_features, n_bins, offs, 256, wg_per_cu)
        assert blocks.shape[0] == int(wgs.sum()) * n_tiles
        seen = set()
        for leaf, tile, wg in blocks.tolist():
            assert 0 <= leaf < n_leaves and 0 <= tile < n_tiles and 0 <= wg < wgs[leaf], (leaf, tile, wg)
            seen.add((leaf, tile, wg))
        assert len(seen) == blocks.shape[0]                      # no (leaf, tile, wg) twice
        for l in range(n_leaves):
            n_epochs = -(-int(sizes[l]) // 512)
            if n_epochs == 0:
                assert wgs[l] == 0
                continue
            # units of 4 epochs, or an even split with one longer unit per workgroup (at most 3 x 4)
            assert 1 <= wgs[l] <= n_epochs and 1 <= ue[l] <= 12
            n_units = -(-n_epochs // int(ue[l]))
            if ue[l] > 4:
                assert n_units == wgs[l]
            assert wgs[l] <= n_units                             # no workgroup without a unit
            # workgroup c takes units c, c + wgs, ...: together all units, each once
            taken = sorted(u for c in range(wgs[l]) for u in range(c, n_units, int(wgs[l])))
            assert taken == list(range(n_units))
        # the longest workgroups start first, to within 1/128 of the longest
        each = [-(-int(sizes[l]) // 512) / wgs[l] if wgs[l] else 0.0 for l in range(n_leaves)]
        starts = list(dict.fromkeys(blocks[blocks[:, 1] == 0][:, 0].tolist()))
        assert all(each[b] <= each[a] + 1 + max(each) / 128 for a, b in zip(starts, starts[1:]))
        # the leaves share the machine: about one machine-full of workgroup columns, plus the
        # at-least-one of every leaf
        assert int(wgs.sum()) <= 256 * wg_per_cu // n_tiles + n_leaves


@pytest.mark.parametrize("n_rows,n_features,n_bins,wg_per_cu,columns",
                         [(8_000_000, 500, 64, 3, 64), (11_000_000, 300, 16, 4, 256), (8_000_000, 500, 256, 2, 64)])
def test_batched_plan_of_equal_leaves_fills_the_cus_evenly(n_rows, n_features, n_bins, wg_per_cu, columns):
    """64 equal leaves: rather one column each, or four, with the same number of workgroups on every CU than a
    second round of columns, or some CUs with one workgroup more than the others."""
    offs = [i * (n_rows // 64) for i in range(65)]
    wgs, _, blocks = B.gbdt_debug_batch_plan(n_features, n_bins, offs, 256, wg_per_cu)
    assert int(wgs.sum()) == columns and len(set(wgs.tolist())) == 1
    assert blocks.shape[0] % 256 == 0


@pytest.mark.parametrize("n_features,n_bins", [(28, 64), (2000, 63), (137, 255), (700, 16)])
def test_wide_accumulation_doubles_the_partial_blocks(n_features, n_bins):
    """The wide mode writes two partial blocks per workgroup; the sizes the library reports for
    caller-owned scratch follow the switch (and go back with it)."""
    n_leaf = 266_000
    narrow = B.gbdt_workspace_bytes(n_leaf, n_features, n_bins)
    narrow_batch = B.gbdt_hist_build_batch_workspace_bytes(n_features, n_bins, 64)
    B.gbdt_set_wide_accumulation(True)
    try:
        wide = B.gbdt_workspace_bytes(n_leaf, n_features, n_bins)
        wide_batch = B.gbdt_hist_build_batch_workspace_bytes(n_features, n_bins, 64)
    finally:
        B.gbdt_set_wide_accumulation(False)
    assert wide >= narrow and wide_batch > narrow_batch
    assert wide_batch <= 2 * narrow_batch
    assert B.gbdt_workspace_bytes(n_leaf, n_features, n_bins) == narrow


def test_fusion_plan_is_a_valid_mixed_radix_packing():
    """Host planner of gbdt_bins_fuse: every feature sits in exactly one column, the levels of a
    column multiply to at most 64, at most 6 features share a column, the weights are the running
    products of the levels in some order of the column's features -- so that a joint value
    decodes back to every feature's bin -- and few-level features really share columns."""
    rng = np.random.default_rng(3)
    for levels in (rng.integers(2, 17, size=700), rng.integers(1, 65, size=333), np.full(40, 2), np.full(9, 64),
                   np.array([1, 1, 1, 64, 33, 2]), rng.integers(1, 5, size=1000)):
        levels = levels.astype(np.uint32)
        col, stride, n_cols = B.gbdt_debug_fusion_plan(levels)
        assert col.min() == 0 and col.max() == n_cols - 1 and len(np.unique(col)) == n_cols
        for c in range(n_cols):
            fs = np.nonzero(col == c)[0]
            assert 1 <= len(fs) <= 6
            assert int(np.prod(levels[fs].astype(np.int64))) <= 64
            order = fs[np.argsort(stride[fs], kind="stable")]
            run = 1
            for f in order:                       # weights: 1, L_a, L_a L_b, ...
                assert stride[f] == run, (c, fs, stride[fs], levels[fs])
                run *= int(levels[f])
            # decode a random joint value
            b = [int(rng.integers(0, levels[f])) for f in fs]
            v = sum(bi * int(stride[f]) for bi, f in zip(b, fs))
            assert v < 64
            assert [(v // int(stride[f])) % int(levels[f]) for f in fs] == b
        # lower bound on columns: the sum of log2(levels) in units of 6 bits
        assert n_cols >= int(np.ceil(np.log2(levels.astype(np.float64)).sum() / 6.0 - 1e-9))
    col, stride, n_cols = B.gbdt_debug_fusion_plan(np.full(40, 2, np.uint32))
    assert n_cols == 7                            # six binary features per column
    col, stride, n_cols = B.gbdt_debug_fusion_plan(np.full(9, 64, np.uint32))
    assert n_cols == 9


def test_fuse_reads_small_matrices_once():
    """Looking at some rows first costs a round trip to the host: not for a matrix that is read in less."""
    assert B.gbdt_debug_fuse_sample_rows(66_000, 8) == 0 and B.gbdt_debug_fuse_sample_rows(1_000_000, 10) == 0
    assert B.gbdt_debug_fuse_sample_rows(60_000, 4000) == 0
    for n_rows, n_features in ((400_000, 2000), (3_000_000, 700), (65_536, 512)):
        assert 0 < B.gbdt_debug_fuse_sample_rows(n_rows, n_features) <= n_rows // 16


@pytest.mark.parametrize("n_bins", [2, 16, 63, 64, 100, 255, 256])
def test_split_search_plan_covers_every_feature(n_bins):
    """The work split of the split search follows the number of histograms of the launch; whatever
    it picks, the steps of all workgroups cover the features, a workgroup has between 1 and 16 wavefronts (the
    kernel's local memory has a place for each) and a step for every one of them, and a launch never has more
    candidates per histogram than a lone histogram (the scratch of gbdt_workspace_bytes is sized by that)."""
    for n_features in (1, 2, 7, 28, 137, 255, 256, 257, 700, 2000, 4000, 20000):
        lone = B.gbdt_debug_split_plan(n_features, n_bins, 1)
        for n_hists in (1, 2, 3, 8, 31, 64, 256, 1024, 32768):
            p = B.gbdt_debug_split_plan(n_features, n_bins, n_hists)
            assert p["group"] >= 1 and p["passes"] >= 1 and p["workgroups"] >= 1
            assert p["group"] == 64 // max(4, 2 ** int(np.ceil(np.log2((n_bins + 3) // 4))))   # (4 bins a lane)
            assert 1 <= p["waves"] <= 16 and p["waves"] <= p["passes"]
            assert p["group"] * p["passes"] * p["workgroups"] >= n_features
            # no workgroup without a feature
            assert p["group"] * p["passes"] * (p["workgroups"] - 1) < n_features
            assert p["workgroups"] <= lone["workgroups"]


LINE_SHAPES = [(1, 64), (40, 255), (32, 255), (64, 256), (96, 200), (100, 255), (137, 255), (64, 63), (70, 64), (100, 64),
               (128, 63), (129, 63), (150, 16), (193, 63), (220, 63), (270, 16), (400, 16), (2000, 63)]
LINE_ROWS = [1, 511, 4095, 4096, 9001, 300_000, 2 ** 25 - 1024, 2 ** 25 - 1023, 40_000_000]


@pytest.mark.parametrize("n_features,n_bins", LINE_SHAPES)
def test_regions_of_tiles(n_features, n_bins):
    """Where the tiles lie: no byte belongs to two of them and all of them to the row bytes, rows of shared regions
    are 128 or 64 bytes of whole lines or the 48 of a lone 32-byte tile and its remainder, and what the build
    reads past the last row is inside the buffer and at 32-bit offsets."""
    g = B.gbdt_debug_geometry(n_features, n_bins, 1)
    widths = [g["wm"]] * g["n_main"] + ([g["wr"]] if g["wr"] else [])
    for n_rows in LINE_ROWS:
        tiles, _ = B.gbdt_debug_block_map(n_features, n_bins, n_rows, 1, False)
        total = B.gbdt_bins_packed_bytes(n_rows, n_features, n_bins)
        regions = {}
        for t, (off, stride) in enumerate(tiles.tolist()):
            assert stride in (widths[t], 128, 64, 48) and off % 16 == 0 and stride % 16 == 0
            base = min(o for o, s in tiles.tolist() if s == stride and o <= off < o + stride)
            regions.setdefault((base, stride), []).append((off - base, widths[t]))
            past = -(-n_rows // 512) * 512          # rows up to the end of the last epoch
            assert past * stride + (off - base) <= 2 ** 32
            assert off + (past - 1) * stride + widths[t] <= total, (n_rows, t)
        at = 0
        for (base, stride), parts in sorted(regions.items()):
            assert base == at                        # regions back to back, their rows filled by their tiles
            assert sorted(parts) == [(sum(w for _, w in sorted(parts)[:i]), sorted(parts)[i][1])
                                     for i in range(len(parts))]
            assert sum(w for _, w in parts) == stride
            at += n_rows * stride
        assert at == n_rows * g["row_bytes"]
        shared = [len(p) > 1 for p in regions.values()]
        assert any(shared) == (4096 <= n_rows <= 2 ** 25 - 1024 and
                               (g["n_main"] >= 2 or (g["wm"] == 32 and len(widths) == 2)))


@pytest.mark.parametrize("n_features,n_bins", LINE_SHAPES)
@pytest.mark.parametrize("by_column", [False, True])
@pytest.mark.parametrize("wide", [False, True])
def test_blocks_of_a_launch(n_features, n_bins, by_column, wide):
    B.gbdt_set_wide_accumulation(wide)
    try:
        check_blocks_of_a_launch(n_features, n_bins, by_column, wide)
    finally:
        B.gbdt_set_wide_accumulation(False)


def check_blocks_of_a_launch(n_features, n_bins, by_column, wide):
    """Every (tile, workgroup) is one block's, whatever the layout; the two tiles of a region get their workgroups of a
    column to the same XCD (blocks 8 apart, except in the last few); a remainder tile of its own comes last; with wide
    accumulation a lone main tile has workgroups all through the launch."""
    g = B.gbdt_debug_geometry(n_features, n_bins, 1)
    n_tiles = g["n_main"] + (1 if g["wr"] else 0)
    for n_rows in (1000, 9001, 2 ** 25):
        for cols in (1, 3, 7, 8, 9, 100, 147, 512):
            tiles, blocks = B.gbdt_debug_block_map(n_features, n_bins, n_rows, cols, by_column)
            at = {tuple(tc): i for i, tc in enumerate(blocks.tolist())}
            assert set(at) == {(t, c) for t in range(n_tiles) for c in range(cols)}
            strides = tiles[:, 1].tolist()
            for t in range(0, n_tiles - 1, 2):
                if strides[t] > g["wm"]:             # (t, t + 1) share a region
                    same = [at[t + 1, c] - at[t, c] for c in range(cols)]
                    assert sum(d != 8 for d in same) <= 7
            lone = g["n_main"] - 1
            if wide and n_rows == 9001 and g["n_main"] % 2 and lone and strides[lone] == g["wm"] and cols >= 16:
                where = np.array(sorted(at[lone, c] for c in range(cols)))
                assert np.diff(where).max() <= 8 * g["n_main"] and where[0] < 8 * g["n_main"]
            if g["wr"] and strides[-1] == g["wr"]:
                assert [at[n_tiles - 1, c] for c in range(cols)] == list(range((n_tiles - 1) * cols, n_tiles * cols))


def test_cell_counts_are_exact_whatever_the_sums_do():
    """A cell's count and sums share 64 bits.  Sums of magnitudes below 2^26 (what the scale of an epoch
    guarantees when the epoch's sum of magnitudes is a finite fp32 number) come back exactly; beyond that, with
    values that a conversion has saturated too, the sums wrap but the count stays exact: tree
    growth finds the rows of a node by its counts."""
    rng = np.random.default_rng(8)
    for trial in range(200):
        n = int(rng.integers(0, 513))
        g, h = (rng.normal(size=n) * (2.0 ** 26 - 257) / max(1, n) / 5 for _ in range(2))
        g, h = np.rint(g).astype(np.int64), np.rint(h).astype(np.int64)
        assert np.abs(g).sum() < 2 ** 26 and np.abs(h).sum() < 2 ** 26
        assert B.gbdt_debug_cell_sums(g, h) == (g.sum(), h.sum(), n)
    top = 2 ** 26 - 257
    for g, h in ((top, -top), (-top, top), (-top, -top), (top, top)):
        assert B.gbdt_debug_cell_sums([g, 0], [0, h]) == (g, h, 2)
    big, small = 2 ** 31 - 1, -2 ** 31
    for g, h in (([big] * 3, [1] * 3), ([small] * 512, [small] * 512), ([big, small, 5], [big, 0, 0]),
                 ([9_860_761] * 7, [0] * 7),        # 1e38 at the smallest scale there is, 2^-103
                 ([0] * 512, [big] * 512), ([-9_860_761] * 100, [9_860_761] * 100)):
        assert B.gbdt_debug_cell_sums(g, h)[2] == len(g), (g[0], h[0])


def test_partition_plan_chunks_cover_the_list():
    """Chunks of 256 * rows_per_thread positions: 8 steps, or a multiple of 16 (the kernels take
    8 or 16 steps at a time), at most 2048 chunks, every position in exactly one chunk."""
    for n in (1, 255, 256, 2047, 2048, 2049, 8192, 8193, 4_194_304, 4_194_305, 10_500_000, 11_000_000,
              67_108_864, 2**31 - 1, 2**32 - 1):
        p = B.gbdt_debug_partition_plan(n)
        r, c = p["rows_per_thread"], p["chunks"]
        assert r == 8 or r % 16 == 0
        assert r & (r - 1) == 0
        assert 1 <= c <= 2048
        assert (c - 1) * 256 * r < n <= c * 256 * r
        assert p["bytes"] == c * r * 4 * 8 + c * 4
    with pytest.raises(B.GbdtError):
        B.gbdt_debug_partition_plan(0)
