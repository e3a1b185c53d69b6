"""The work that a gradient-boosting trainer has this library do, as cases for a benchmark.

A trainer bins its data once and packs it (`load`), and then, for every tree, builds histograms of
leaves, forms siblings by subtraction, searches splits and partitions rows -- itself, one leaf at a
time (`step`) or a level at a time (`level`, `search`), or by the library's own growers (`tree`,
`tree_depth`).  The shapes are those of synth.py's five workloads and of the paper's kernel
benchmark (8,000,000 x 500 uniform bins, App. C.2); `draw` covers the ranges between them.

Gradients and hessians are those of the logistic loss.  Histograms are compared as numbers.  A
whole tree can only be compared when no choice among its splits hangs on a rounding, so trees are
grown from the gradients of the first boosting iteration (all scores zero: +-1/2 and 1/4), whose
sums every correct implementation has exactly.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1706_08359_amd import binding as B
from paper_1706_08359_amd import synth

LAM, MIN_CHILD_HESS = 1.0, 1e-3


def listed():
    return [
        # the smallest calls: the root of 10,000 x 28 with 64 bins; latency and launches
        dict(name="tiny_step", kind="step", rows=10_000, features=28, bins=64, data="uniform", left=0.0, wide=False),
        # the root of the epsilon-shaped matrix, the shape the headline number is quoted on
        dict(name="dense_wide_step", kind="step", rows=400_000, features=2000, bins=63, data="uniform", left=0.0,
             wide=False),
        # the root of the Higgs-shaped matrix: few features, 255 bins, one tile
        dict(name="dense_tall_step", kind="step", rows=10_500_000, features=28, bins=255, data="uniform", left=0.0,
             wide=False),
        # a quarter of the rows of the ranking matrix (60 % zeros): one split of the root
        dict(name="ranking_leaf", kind="step", rows=2_270_000, features=137, bins=255, data="uniform_zeros",
             left=0.25, wide=False),
        # few-level features: 4-bit bins, columns shared by several features
        dict(name="categorical_step", kind="step", rows=3_000_000, features=700, bins=16, data="levels", left=0.0,
             wide=False),
        # a leaf of an eighth of the rows of the paper's benchmark matrix (depth 3)
        dict(name="paper_leaf", kind="step", rows=8_000_000, features=500, bins=64, data="uniform", left=0.125,
             wide=False),
        # the double precision switch, on the ranking matrix's root
        dict(name="ranking_wide_sums", kind="step", rows=2_270_000, features=137, bins=255, data="uniform_zeros",
             left=0.0, wide=True),
        # one level of a tree in two calls: 64 leaves of unequal size
        dict(name="level_64", kind="level", rows=1_500_000, features=500, bins=255, data="uniform", depth=6),
        # the splits of a level's 64 histograms in one call
        dict(name="search_64", kind="search", rows=400_000, features=2000, bins=63, hists=64),
        # a whole tree, leaf-wise, with the paper's 255 leaves
        dict(name="tree_tall", kind="tree", rows=10_500_000, features=28, bins=255, data="uniform", leaves=255),
        # a whole tree, level-wise, depth 8
        dict(name="tree_depth_wide", kind="tree_depth", rows=400_000, features=2000, bins=63, data="uniform", depth=8),
        # what comes before the first tree: packing the binned matrix, the root, its split and its rows
        dict(name="load_wide", kind="load", rows=400_000, features=2000, bins=63, data="uniform"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, most_values, rows_lo=2_000, rows_hi=10_500_000, features_hi=2000):
    """rows, features, bins and data of a matrix of at most most_values values."""
    features = _log_int(rng, 4, features_hi)
    rows = _log_int(rng, rows_lo, min(rows_hi, most_values // features))
    cap = rng.choice([16, 64, 64, 256, 256])
    if cap == 16:
        return rows, features, rng.randint(4, 16), "levels"
    bins = rng.randint(24, 64) if cap == 64 else rng.randint(100, 256)
    return rows, features, bins, rng.choice(["uniform", "uniform", "uniform_zeros"])


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "level", "search", "tree", "tree_depth", "load"])
    if kind == "search":
        features, bins, hists = _log_int(rng, 4, 2000), rng.randint(4, 256), _log_int(rng, 1, 128)
        while hists * features * bins > 64 * 2000 * 63:
            hists = max(1, hists // 2)
        return dict(kind=kind, rows=_log_int(rng, 50_000, 10_000_000), features=features, bins=bins, hists=hists)
    most = {"step": 1_000_000_000, "level": 600_000_000, "tree": 290_000_000, "tree_depth": 400_000_000,
            "load": 700_000_000}[kind]
    rows, features, bins, data = _shape(rng, most, rows_lo=2_000 if kind in ("step", "load") else 10_000)
    case = dict(kind=kind, rows=rows, features=features, bins=bins, data=data)
    if kind == "step":
        case["left"] = 0.0 if rng.random() < 0.4 else math.exp(rng.uniform(math.log(0.02), math.log(0.5)))
        case["wide"] = rng.random() < 0.2
    elif kind == "level":
        case["depth"] = rng.randint(1, 7)
    elif kind == "tree":
        case["leaves"] = rng.choice([15, 31, 63, 127, 255])
    elif kind == "tree_depth":
        case["depth"] = rng.randint(3, 8)
    return case


# --------------------------------------------------------------------------- inputs


def _matrix(case, gen):
    """uint8 [rows, features] on the GPU."""
    n, f, nb = case["rows"], case["features"], case["bins"]
    if case["data"] == "uniform":          # quantile bins of any continuous feature
        return synth.uniform_bins(n, f, nb, gen, "cuda")
    out = torch.empty((n, f), dtype=torch.uint8, device="cuda")
    step = max(1, (1 << 28) // f)
    if case["data"] == "uniform_zeros":    # 60 % zeros in bin 0, quantile bins of the rest
        for r in range(0, n, step):
            m = min(n, r + step) - r
            nz = torch.randint(1, nb, (m, f), generator=gen, device="cuda", dtype=torch.uint8)
            hundred = torch.randint(0, 100, (m, f), generator=gen, device="cuda", dtype=torch.uint8)
            out[r:r + m] = torch.where(hundred < 60, torch.zeros_like(nz), nz)
        return out
    # "levels": every feature has 2 .. nb levels, low levels more often (min of two uniform draws)
    levels = torch.randint(2, nb + 1, (f,), generator=gen, device="cuda").to(torch.int16)
    for r in range(0, n, step):
        m = min(n, r + step) - r
        a = torch.randint(0, 240, (m, f), generator=gen, device="cuda", dtype=torch.uint8)
        b = torch.randint(0, 240, (m, f), generator=gen, device="cuda", dtype=torch.uint8)
        u = torch.minimum(a, b).to(torch.int16)
        out[r:r + m] = torch.div(u * levels, 240, rounding_mode="floor").to(torch.uint8)
    return out


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _threshold(bins, feature, left):
    """The threshold of `feature` that sends a share of rows closest to `left` to the left, and that many rows."""
    counts = torch.bincount(bins[:, feature].to(torch.int64), minlength=2)
    cum = torch.cumsum(counts, 0)[:-1].clamp(min=1)
    thr = int(torch.argmin((cum.double() / bins.shape[0] - left).abs()).item())
    return thr, int(counts[:thr + 1].sum().item())


def _step_inputs(case, seed):
    gen = _gen(seed)
    bins = _matrix(case, gen)
    grad, hess = synth.logistic_grad_hess(case["rows"], gen, "cuda", score_std=0.1)
    feature, thr, n_left = case["features"] // 2, 0, 0
    if case["left"] > 0.0:
        thr, n_left = _threshold(bins, feature, case["left"])
    return bins, grad, hess, feature, thr, n_left


def _level_inputs(case, seed):
    """A level of a tree: the rows of its 2^depth leaves back to back (ascending inside a leaf), and each
    leaf's split (feature, threshold)."""
    gen = _gen(seed)
    bins = _matrix(case, gen)
    grad, hess = synth.logistic_grad_hess(case["rows"], gen, "cuda", score_std=0.1)
    leaf = torch.zeros(case["rows"], dtype=torch.int32, device="cuda")
    for d in range(case["depth"]):  # the way down: one column per level, cut a little off its middle
        col = bins[:, d % case["features"]]
        leaf = 2 * leaf + (col > int(case["bins"] * (0.3 if d % 2 else 0.45))).to(torch.int32)
    n_leaves = 1 << case["depth"]
    row_idx = torch.sort(leaf, stable=True).indices.to(torch.int32)
    sizes = torch.bincount(leaf.to(torch.int64), minlength=n_leaves).tolist()
    offsets = [0]
    for s in sizes:
        offsets.append(offsets[-1] + s)
    features = torch.randint(0, case["features"], (n_leaves,), generator=gen, device="cuda").tolist()
    splits = torch.cat([B.split_record(f, int(case["bins"] * (0.3 + 0.01 * (i % 40))), "cuda").reshape(1, 9)
                        for i, f in enumerate(features)])
    return bins, grad, hess, row_idx, offsets, splits


def _search_inputs(case, seed):
    """Histograms of a level: counts around rows / (hists * bins), sums of logistic gradients over them."""
    gen = _gen(seed)
    shape = (case["hists"], case["features"], case["bins"])
    mean = max(1.0, case["rows"] / (case["hists"] * case["bins"]))
    noise = torch.randn(shape, generator=gen, device="cuda")
    count = (mean + noise * math.sqrt(mean)).round().clamp(min=0.0)
    drift = torch.linspace(-0.02, 0.02, case["bins"], device="cuda")
    grad = 0.5 * count.sqrt() * torch.randn(shape, generator=gen, device="cuda") + count * drift
    hess = count * (0.2475 + 0.001 * torch.rand(shape, generator=gen, device="cuda"))
    hists = torch.empty(shape + (3,), dtype=torch.float32, device="cuda")
    hists[..., 0], hists[..., 1] = grad, hess
    hists.view(torch.int32)[..., 2] = count.to(torch.int32)
    return hists


def _pack(bins, case):
    return B.gbdt_bins_pack(bins, case["bins"])


def _hist_views(hist):
    """The sums and the counts of histograms as two tensors on the same memory."""
    return hist[..., :2], hist.view(torch.int32)[..., 2]


def _split_views(rec):
    """(feature, bin), (gain, left sums, right sums) and the counts of split records."""
    f = rec.view(torch.float32)
    return rec[:, :2], f[:, 2:5], f[:, 6:8], rec[:, 5::3]


def prepare(case, seed):
    kind, n, f, nb = case["kind"], case["rows"], case["features"], case["bins"]
    st = dict(case=dict(case))

    def hist_buffer(*lead):
        return torch.empty(lead + (f, nb, 3), dtype=torch.float32, device="cuda")

    def split_buffer(k):
        return torch.empty((k, 9), dtype=torch.int32, device="cuda")

    if kind == "search":
        st.update(hists=_search_inputs(case, seed), rec=split_buffer(case["hists"]))
        st["out"] = _split_views(st["rec"])
        return st
    if kind in ("step", "load"):
        bins, grad, hess, feature, thr, n_left = _step_inputs(dict(case, left=case.get("left", 0.0)), seed)
        st.update(grad=grad, hess=hess, hist=hist_buffer(), rec=split_buffer(1))
        st["out"] = _hist_views(st["hist"]) + _split_views(st["rec"])
        if kind == "load":
            st.update(bins=bins, packed=torch.zeros(B.gbdt_bins_packed_bytes(n, f, nb), dtype=torch.uint8,
                                                    device="cuda"),
                      split=B.split_record(f // 3, nb // 2, "cuda"))
            st["children"] = torch.empty(n, dtype=torch.int32, device="cuda")
            st["n_left"] = torch.empty(1, dtype=torch.int64, device="cuda")
            st["out"] += (st["children"], st["n_left"])
            return st
        st["packed"] = _pack(bins, case)
        if n_left:
            st.update(split=B.split_record(feature, thr, "cuda"), n_of_leaf=n_left,
                      parent=B.gbdt_hist_build(st["packed"], n, f, nb, None, n, grad, hess),
                      sibling=hist_buffer())
            st["children"] = torch.empty(n, dtype=torch.int32, device="cuda")
            st["n_left"] = torch.empty(1, dtype=torch.int64, device="cuda")
            st["out"] += _hist_views(st["sibling"]) + (st["children"], st["n_left"])
        return st
    if kind == "level":
        bins, grad, hess, row_idx, offsets, splits = _level_inputs(case, seed)
        st.update(packed=_pack(bins, case), grad=grad, hess=hess, row_idx=row_idx, offsets=offsets, splits=splits,
                  hist=hist_buffer(len(offsets) - 1), children=torch.empty_like(row_idx),
                  n_left=torch.empty(len(offsets) - 1, dtype=torch.int64, device="cuda"))
        st["out"] = _hist_views(st["hist"]) + (st["children"], st["n_left"])
        return st
    gen = _gen(seed)                                         # the growers
    bins = _matrix(case, gen)
    grad, hess = synth.labels_with_signal(bins, nb, gen)     # scores zero: +-1/2 and 1/4
    st.update(packed=_pack(bins, case), grad=grad, hess=hess,
              rows_out=torch.empty(n, dtype=torch.int32, device="cuda"))
    st["most_nodes"] = 2 * case["leaves"] - 1 if kind == "tree" else 2 ** (case["depth"] + 1) - 1
    if kind == "tree":
        need = B.gbdt_grow_tree_scratch_bytes(n, f, nb, case["leaves"])
    else:
        need = int(B.load().gbdt_grow_tree_depthwise_scratch_bytes(n, f, nb, case["depth"]))
    st["scratch"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return st


def run(st):
    case = st["case"]
    kind, n, f, nb = case["kind"], case["rows"], case["features"], case["bins"]
    if kind == "step":
        if case["wide"]:
            B.gbdt_set_wide_accumulation(True)
        if "parent" in st:   # one split of the root: its rows, the left child, the right one by subtraction
            B.gbdt_partition_rows(st["packed"], n, f, nb, None, n, st["split"], children_out=st["children"],
                                  n_left_out=st["n_left"])
            B.gbdt_hist_build(st["packed"], n, f, nb, st["children"], st["n_of_leaf"], st["grad"], st["hess"],
                              hist_out=st["hist"])
            B.gbdt_hist_subtract(st["parent"], st["hist"], sibling_out=st["sibling"])
        else:
            B.gbdt_hist_build(st["packed"], n, f, nb, None, n, st["grad"], st["hess"], hist_out=st["hist"])
        B.gbdt_best_split(st["hist"], LAM, MIN_CHILD_HESS, split_out=st["rec"])
        if case["wide"]:
            B.gbdt_set_wide_accumulation(False)
        return st["out"]
    if kind == "level":
        B.gbdt_hist_build_batch(st["packed"], n, f, nb, st["row_idx"], st["offsets"], st["grad"], st["hess"],
                                hist_out=st["hist"])
        B.gbdt_partition_rows_batch(st["packed"], n, f, nb, st["row_idx"], st["offsets"], st["splits"],
                                    children_out=st["children"], n_left_out=st["n_left"])
        return st["out"]
    if kind == "search":
        B.gbdt_best_split_batch(st["hists"], LAM, MIN_CHILD_HESS, splits_out=st["rec"])
        return st["out"]
    if kind == "load":
        B.gbdt_bins_pack(st["bins"], nb, packed_out=st["packed"])
        B.gbdt_hist_build(st["packed"], n, f, nb, None, n, st["grad"], st["hess"], hist_out=st["hist"])
        B.gbdt_best_split(st["hist"], LAM, MIN_CHILD_HESS, split_out=st["rec"])
        B.gbdt_partition_rows(st["packed"], n, f, nb, None, n, st["split"], children_out=st["children"],
                              n_left_out=st["n_left"])
        return st["out"]
    if kind == "tree":
        nodes, order, _ = B.gbdt_grow_tree(st["packed"], n, f, nb, st["grad"], st["hess"], case["leaves"], LAM,
                                           MIN_CHILD_HESS, 0.0, scratch=st["scratch"], row_order_out=st["rows_out"])
    else:
        nodes, order, _ = B.gbdt_grow_tree_depthwise(st["packed"], n, f, nb, st["grad"], st["hess"], case["depth"],
                                                     LAM, MIN_CHILD_HESS, 0.0, scratch=st["scratch"],
                                                     row_order_out=st["rows_out"])
    tree = np.zeros(st["most_nodes"], dtype=nodes.dtype)   # a model keeps its trees in arrays of one size
    tree[:len(nodes)] = nodes
    return {"rows": order, **{k: tree[k] for k in tree.dtype.names if k != "reserved"}}


def work(case):
    kind, n, f, nb = case["kind"], case["rows"], case["features"], case["bins"]
    hist = f * nb * 12
    bpv = 0.5 if nb <= 16 else 1.0
    if kind == "search":
        return {"bytes": case["hists"] * (hist + 36), "flops": case["hists"] * f * nb * 12}
    if kind == "step":
        if case["left"] <= 0.0:
            return {"bytes": n * f * bpv + 8 * n + hist + 36, "flops": 2 * n * f}
        m = max(1, int(n * case["left"]))
        # the split column and the two lists, then the child's rows, the parent read and two histograms written
        return {"bytes": n + 4 * n + m * (f * bpv + 12) + 3 * hist + 36, "flops": 2 * m * f}
    if kind == "level":
        return {"bytes": n * f * bpv + 12 * n + (1 << case["depth"]) * hist + 9 * n, "flops": 2 * n * f}
    if kind == "load":  # the matrix read, the tiles and the columns written; the root; its rows
        return {"bytes": n * f * (2 + bpv) + n * f * bpv + 8 * n + hist + 5 * n, "flops": 2 * n * f}
    # a tree: the root, then per level of a balanced tree every row once in a partition and half of the rows in
    # the smaller children's histograms; a histogram per node
    levels = case["depth"] if kind == "tree_depth" else max(1.0, math.log2(case["leaves"]))
    nodes = 2 ** levels
    return {"bytes": n * f * bpv + 8 * n + levels * (9 * n + n / 2 * (f * bpv + 12)) + 3 * nodes * hist,
            "flops": 2 * n * f * (1 + levels / 2)}


def tolerance(case):
    """Trees are compared from exact sums (see above), searches from the same histograms: only the fp32 rounding of
    a gain is left.  Sums of histograms, against 64 bits over these ranges: up to 2e-6 of the norm and 4.5e-5 at one
    bin (few rows and many bins); with wide accumulation 3e-8 and 6e-8, and for siblings (the difference of two
    rounded sums) 2.4e-7 and 1.6e-6.  Four times that is allowed."""
    if case["kind"] in ("tree", "tree_depth", "search"):
        return {"rel": 1e-6, "max": 1e-5}
    if case.get("wide"):
        return {"rel": 1e-6, "max": 6e-6}
    return {"rel": 8e-6, "max": 1.8e-4}


# --------------------------------------------------------------------------- in 64 bits


def _exact_hist(bins, nb, grad, hess, row_idx=None):
    """float64 [features, bins, 3]: the sums of grad, hess and 1 over the rows row_idx (all: None).  Rows take turns
    in a number of copies, so that a frequent bin is not one address that all of them wait for."""
    f = bins.shape[1]
    copies = max(1, min(64, (1 << 24) // (f * nb)))
    out = torch.zeros((copies * f * nb, 3), dtype=torch.float64, device="cuda")
    base = torch.arange(f, device="cuda", dtype=torch.int64) * nb
    n = bins.shape[0] if row_idx is None else row_idx.numel()
    step = max(1, (1 << 24) // f)
    for r in range(0, n, step):
        if row_idx is None:
            b, g, h = bins[r:r + step], grad[r:r + step], hess[r:r + step]
        else:
            rows = row_idx[r:r + step].to(torch.int64)
            b, g, h = bins[rows], grad[rows], hess[rows]
        copy = (torch.arange(b.shape[0], device="cuda") % copies) * (f * nb)
        at = (b.to(torch.int64) + base + copy[:, None]).reshape(-1)
        v = torch.stack([g.double(), h.double(), torch.ones_like(g, dtype=torch.float64)], dim=1)
        out.index_add_(0, at, v[:, None, :].expand(-1, f, -1).reshape(-1, 3))
    return out.reshape(copies, f, nb, 3).sum(dim=0)


def _exact_split(sums, counts):
    """(gain, left sums), (right sums) of the best split of [hists, features, bins, 2] sums, in 64 bits."""
    p, c = torch.cumsum(sums, dim=2), torch.cumsum(counts, dim=2)
    tot, n = p[:, :, -1:, :], c[:, :, -1:]
    gl, hl = p[..., 0], p[..., 1]
    gr, hr = tot[..., 0] - gl, tot[..., 1] - hl
    gain = gl * gl / (hl + LAM) + gr * gr / (hr + LAM) - tot[..., 0] ** 2 / (tot[..., 1] + LAM)
    ok = (c >= 1) & (n - c >= 1) & (hl >= MIN_CHILD_HESS) & (hr >= MIN_CHILD_HESS)
    gain = torch.where(ok, gain, torch.full_like(gain, -math.inf))[:, :, :-1].reshape(sums.shape[0], -1)
    best = gain.argmax(dim=1)
    f, t = best // (sums.shape[2] - 1), best % (sums.shape[2] - 1)
    k = torch.arange(sums.shape[0], device="cuda")
    left = torch.stack([gain[k, best], gl[k, f, t], hl[k, f, t]], dim=1)
    return left, torch.stack([gr[k, f, t], hr[k, f, t]], dim=1)


def exact(case, seed):
    kind, nb = case["kind"], case["bins"]
    if kind in ("tree", "tree_depth"):
        return None  # a whole tree in plain torch takes minutes
    if kind == "search":
        hists = _search_inputs(case, seed)
        left, right = _exact_split(hists[..., :2].double(), hists.view(torch.int32)[..., 2].double())
        return None, left, right, None
    if kind == "level":
        bins, grad, hess, row_idx, offsets, _ = _level_inputs(case, seed)
        hists = [_exact_hist(bins, nb, grad, hess, row_idx[a:b])[..., :2] for a, b in zip(offsets, offsets[1:])]
        return torch.stack(hists), None, None, None
    bins, grad, hess, feature, thr, n_left = _step_inputs(dict(case, left=case.get("left", 0.0)), seed)
    rows = torch.nonzero(bins[:, feature] <= thr).reshape(-1) if n_left else None
    hist = _exact_hist(bins, nb, grad, hess, rows)
    left, right = _exact_split(hist[None, ..., :2], hist[None, ..., 2])
    out = (hist[..., :2], None, None, left, right, None)
    if n_left:
        out += ((_exact_hist(bins, nb, grad, hess) - hist)[..., :2], None, None, None)
    elif kind == "load":
        out += (None, None)
    return out
