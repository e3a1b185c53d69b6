"""Feature tiles that share the rows of one region (two 64-byte or two 32-byte tiles a row, and the
tiles that are left over together): every combination of whole lines, a lone main tile and a remainder
tile, on both sides of the row count from which tiles share rows, built as a root, as an index list, in a
batch with empty, short and long leaves, and partitioned by a feature of every tile; dealt out by lines and not;
long leaves whose workgroups start with a long unit.

The gradients are multiples of 1/2 and the hessians of 1/4, so every sum is exact and has to agree
with the oracle bit for bit."""
import numpy as np
import pytest
import torch

from oracle import gbdt_oracle as orc
from paper_1706_08359_amd import binding as B
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu

# features: 64 bins 1 main + remainder, 2 main, 3 main, 3 main + remainder; 255 bins the same with
# 32-byte tiles, and one short of a whole line; 16 bins with two features a byte
SHAPES = [(70, 64), (128, 63), (190, 64), (210, 40), (40, 255), (64, 256), (96, 200), (63, 255), (137, 255),
          (270, 16), (385, 7)]
ROWS = [4095, 4096, 9001]


def problem(n_rows, n_features, n_bins, seed=5):
    rng = np.random.default_rng(seed + n_rows + n_features)
    bins = rng.integers(0, n_bins, size=(n_rows, n_features)).astype(np.uint8)
    grad = (rng.integers(-2, 3, size=n_rows) * 0.5).astype(np.float32)
    hess = (rng.integers(1, 4, size=n_rows) * 0.25).astype(np.float32)
    return GpuProblem(bins, n_bins, grad, hess), rng


def same(got_t, ref, what):
    got = B.hist_to_numpy(got_t)
    for k in ("grad", "hess", "count"):
        assert np.array_equal(got[k].astype(np.float64), ref[k].astype(np.float64)), (what, k)


@pytest.mark.parametrize("n_features,n_bins", SHAPES)
@pytest.mark.parametrize("n_rows", ROWS)
def test_lines_of_tiles(n_rows, n_features, n_bins):
    print(f"lines {n_rows} x {n_features}, {n_bins} bins", flush=True)
    p, rng = problem(n_rows, n_features, n_bins)
    same(p.build(), p.oracle(), "root")
    same(p.build(n_leaf=n_rows - 511), p.oracle(n_leaf=n_rows - 511), "first rows")
    idx = np.sort(rng.choice(n_rows, size=n_rows // 3, replace=False)).astype(np.int32)
    same(p.build(idx), p.oracle(idx), "list")
    sizes = [0, 1, 513, n_rows // 2, 0, 2100]
    perm = np.concatenate([np.sort(rng.choice(n_rows, size=s, replace=False)) for s in sizes]).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(sizes)])
    hists = B.gbdt_hist_build_batch(p.packed, n_rows, n_features, n_bins, torch.from_numpy(perm).to(p.dev), offs,
                                    p.grad, p.hess)
    for l in range(len(sizes)):
        same(hists[l], p.oracle(perm[offs[l]:offs[l + 1]]), f"leaf {l}")
    # the short-list partition reads the tiles: one feature of the first and last tile, one in between
    bins = p.bins_cpu.numpy()
    for f in (0, n_features // 2, n_features - 1):
        rec = B.split_record(f, n_bins // 2, p.dev)
        kids, n_left = B.gbdt_partition_rows(p.packed, n_rows, n_features, n_bins, torch.from_numpy(idx).to(p.dev),
                                             idx.size, rec)
        left, right = orc.partition_rows(bins, f, n_bins // 2, idx)
        assert int(n_left.item()) == left.size
        assert np.array_equal(kids.cpu().numpy()[:idx.size], np.concatenate([left, right])), f


def rows_for(n_features, n_bins, epochs_each):
    """Rows of a root that gives every workgroup `epochs_each` epochs on this device, wide accumulation or not."""
    tiles, _ = B.gbdt_debug_block_map(n_features, n_bins, 1, 1, False)
    g = B.gbdt_debug_geometry(n_features, n_bins, 1)
    most = max(B.gbdt_debug_occupancy(g["cap"], i) for i in (False, True))
    n_cus = torch.cuda.get_device_properties(0).multi_processor_count
    return int(most * n_cus // len(tiles) * epochs_each * 512) + 1


def check_features(p, got_t, feats, idx, what):
    got = B.hist_to_numpy(got_t)
    ref = p.oracle(idx, features=feats)
    for j, f in enumerate(feats):
        for k in ("grad", "hess", "count"):
            assert np.array_equal(got[k][f].astype(np.float64), ref[k][j].astype(np.float64)), (what, f, k)


@pytest.mark.parametrize("n_features,n_bins", SHAPES)
def test_lines_of_tiles_dealt_out(n_features, n_bins):
    """Leaves of two or three epochs a workgroup: the blocks are dealt out by shared lines (shorter leaves, as above, are
    not), the first and last feature of every tile checked."""
    n_rows = rows_for(n_features, n_bins, 2.5)
    print(f"dealt {n_rows} x {n_features}, {n_bins} bins", flush=True)
    plan = B.gbdt_debug_leaf_plan(n_rows, n_features, n_bins, n_rows, False)
    assert plan["deal"] == 1 and plan["unit_epochs"] in (2, 3)
    p, rng = problem(n_rows, n_features, n_bins)
    first = {}
    for f in range(n_features):
        first.setdefault(B.gbdt_debug_locate(n_features, n_bins, f)[0], []).append(f)
    feats = sorted({f for fs in first.values() for f in (fs[0], fs[-1])})
    check_features(p, p.build(), feats, None, "root")
    idx = np.sort(rng.choice(n_rows, size=n_rows - n_rows // 8, replace=False)).astype(np.int32)
    check_features(p, p.build(idx), feats, idx, "list")
    offs = np.array([0, n_rows // 3, n_rows // 3, n_rows // 3 + 5, idx.size])
    perm = np.concatenate([np.sort(part) for part in np.split(rng.permutation(idx), offs[1:-1])]).astype(np.int32)
    wgs, ue, _ = B.gbdt_debug_batch_plan(n_features, n_bins, offs, 256, B.gbdt_debug_occupancy(n_bins, True))
    assert ue.max() > 1
    hists = B.gbdt_hist_build_batch(p.packed, n_rows, n_features, n_bins, torch.from_numpy(perm).to(p.dev), offs,
                                    p.grad, p.hess)
    for l in range(len(offs) - 1):
        check_features(p, hists[l], feats, perm[offs[l]:offs[l + 1]], f"leaf {l}")


@pytest.mark.parametrize("n_features,n_bins", [(210, 63), (137, 255), (270, 16)])
def test_long_leaf_starts_with_long_units(n_features, n_bins):
    """Enough epochs that every workgroup starts with one long unit and takes short ones after it, with
    rows at the very end of the leaf, as a root and as a list, in the default mode, in the bit-reproducible one (one
    even unit each) and with wide accumulation."""
    n_rows = rows_for(n_features, n_bins, 16)
    print(f"long leaf {n_rows} x {n_features}, {n_bins} bins", flush=True)
    p, rng = problem(n_rows, n_features, n_bins)
    feats = [0, n_features // 2, n_features - 1]
    idx = np.nonzero(rng.random(n_rows) < 0.9)[0].astype(np.int32)
    idx[-1] = n_rows - 1
    for det, wide in ((False, False), (True, False), (False, True), (True, True)):
        B.gbdt_set_deterministic(det)
        B.gbdt_set_wide_accumulation(wide)
        try:
            for rows in (None, idx):
                n_leaf = n_rows if rows is None else rows.size
                plan = B.gbdt_debug_leaf_plan(n_rows, n_features, n_bins, n_leaf, rows is not None)
                n_epochs = -(-n_leaf // 512)
                assert plan["one_unit_each"] == 0 and plan["deal"] == (2 if wide else 1)
                if det:
                    assert plan["first_epochs"] == 0 and plan["fixed_stride"] == plan["wgs"]
                    assert plan["unit_epochs"] == -(-n_epochs // plan["wgs"])
                else:
                    assert plan["first_epochs"] >= 4 and plan["fixed_stride"] == 0 and plan["unit_epochs"] >= 3
                    assert plan["first_epochs"] * plan["wgs"] < n_epochs
                check_features(p, p.build(rows), feats, rows, (det, wide, rows is None))
        finally:
            B.gbdt_set_deterministic(False)
            B.gbdt_set_wide_accumulation(False)


@pytest.mark.parametrize("n_rows", [2 ** 25 - 1024, 2 ** 25 - 1023])
def test_largest_shared_regions(n_rows):
    """The last row count whose byte offsets in a region of 128-byte rows fit 32 bits, and the first with a region per
    tile: the root, a list with the last rows, and the short-list partition by a feature of the second tile.
    (97 features of one byte are two tiles of 64; the reference is computed on the device, from exact sums.)"""
    F, nb, dev = 97, 64, torch.device("cuda:0")
    print(f"largest regions {n_rows} x {F}", flush=True)
    tiles, _ = B.gbdt_debug_block_map(F, nb, n_rows, 1, False)
    assert tiles[:, 1].tolist() == ([128, 128] if n_rows == 2 ** 25 - 1024 else [64, 64])
    gen = torch.Generator(device=dev)
    gen.manual_seed(4)
    bins = torch.randint(0, nb, (n_rows, F), generator=gen, device=dev, dtype=torch.uint8)
    grad = torch.randint(-2, 3, (n_rows,), generator=gen, device=dev).float() * 0.5
    hess = torch.randint(1, 4, (n_rows,), generator=gen, device=dev).float() * 0.25
    packed = B.gbdt_bins_pack(bins, nb, fuse=False)
    idx = torch.cat([torch.randperm(n_rows - 3000, generator=gen, device=dev)[:150_000].sort().values,
                     torch.arange(n_rows - 3000, n_rows, device=dev)]).to(torch.int32)
    for rows in (None, idx):
        n_leaf = n_rows if rows is None else rows.numel()
        got = B.gbdt_hist_build(packed, n_rows, F, nb, rows, n_leaf, grad, hess)
        for f in (0, 63, 64, 96):
            col = bins[:, f] if rows is None else bins[rows.long(), f]
            g, h = (grad, hess) if rows is None else (grad[rows.long()], hess[rows.long()])
            for b in range(nb):
                at = col == b
                assert int(got.view(torch.int32)[f, b, 2]) == int(at.sum()), (f, b)
                assert float(got[f, b, 0]) == float(g[at].sum(dtype=torch.float64)), (f, b)
                assert float(got[f, b, 1]) == float(h[at].sum(dtype=torch.float64)), (f, b)
    short = idx[-6000:].contiguous()
    for f in (63, 64, 96):
        kids, n_left = B.gbdt_partition_rows(packed, n_rows, F, nb, short, short.numel(), B.split_record(f, 30, dev))
        left = bins[short.long(), f] <= 30
        assert int(n_left) == int(left.sum())
        assert torch.equal(kids[:short.numel()], torch.cat([short[left], short[~left]]))


def test_long_list_of_a_lone_tile():
    """A list whose tiles share no lines takes units of four epochs from the start, a root of the same rows does not."""
    n_features, n_bins = 20, 64
    n_rows = rows_for(n_features, n_bins, 15)
    print(f"long list {n_rows} x {n_features}", flush=True)
    p, rng = problem(n_rows, n_features, n_bins)
    idx = np.nonzero(rng.random(n_rows) < 0.95)[0].astype(np.int32)
    for rows in (None, idx):
        n_leaf = n_rows if rows is None else rows.size
        plan = B.gbdt_debug_leaf_plan(n_rows, n_features, n_bins, n_leaf, rows is not None)
        assert plan["one_unit_each"] == 0 and plan["fixed_stride"] == 0
        assert (plan["first_epochs"], plan["unit_epochs"]) == (0, 4) if rows is not None else plan["first_epochs"] >= 4
        check_features(p, p.build(rows), [0, 7, 19], rows, rows is None)
