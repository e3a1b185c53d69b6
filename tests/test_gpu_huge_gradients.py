"""Finite gradients whose sum of magnitudes over an epoch of rows is past the largest fp32 number: the sums of a
bin cannot be represented, but every count is exact, and so the growers, which find the rows of a node by its
counts, give every row to exactly one leaf."""
import numpy as np
import pytest
import torch

from oracle import gbdt_oracle as orc
from paper_1706_08359_amd import binding as B
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu


def problem(n_rows, n_features, n_bins):
    rng = np.random.default_rng(n_rows + n_bins)
    bins = rng.integers(0, n_bins, size=(n_rows, n_features)).astype(np.uint8)
    grad = rng.choice(np.array([1e38, -1e38, 3e38], np.float32), size=n_rows)
    hess = rng.choice(np.array([1e38, 2e38], np.float32), size=n_rows)
    return GpuProblem(bins, n_bins, grad, hess), rng


@pytest.mark.parametrize("n_features,n_bins", [(40, 16), (70, 63), (40, 255)])
@pytest.mark.parametrize("wide", [False, True])
def test_counts_of_huge_gradients(n_features, n_bins, wide):
    n_rows = 20_011
    print(f"huge gradients {n_rows} x {n_features}, {n_bins} bins, wide {wide}", flush=True)
    p, rng = problem(n_rows, n_features, n_bins)
    idx = np.sort(rng.choice(n_rows, size=7001, replace=False)).astype(np.int32)
    sizes = [3, 700, 6298]
    offs = np.concatenate([[0], np.cumsum(sizes)])
    B.gbdt_set_wide_accumulation(wide)
    try:
        root, child = p.build(), p.build(idx)
        batch = B.gbdt_hist_build_batch(p.packed, n_rows, n_features, n_bins, torch.from_numpy(idx).to(p.dev), offs,
                                        p.grad, p.hess)
    finally:
        B.gbdt_set_wide_accumulation(False)
    bins = p.bins_cpu.numpy()
    one = np.ones(n_rows, np.float32)
    for got, rows in [(root, None), (child, idx)] + [(batch[l], idx[offs[l]:offs[l + 1]]) for l in range(len(sizes))]:
        ref = orc.hist_build(bins, n_bins, one, one, rows)
        assert np.array_equal(B.hist_to_numpy(got)["count"].astype(np.uint64), ref["count"])


@pytest.mark.parametrize("n_features,n_bins", [(40, 16), (28, 64), (40, 255)])
@pytest.mark.parametrize("grower", ["leafwise", "depthwise"])
def test_rows_of_trees_on_huge_gradients(n_features, n_bins, grower):
    n_rows = 9001
    print(f"tree on huge gradients {grower} {n_rows} x {n_features}, {n_bins} bins", flush=True)
    p, _ = problem(n_rows, n_features, n_bins)
    if grower == "leafwise":
        nodes, order, _ = B.gbdt_grow_tree(p.packed, n_rows, n_features, n_bins, p.grad, p.hess, 15, 1.0, 1e-3)
    else:
        nodes, order, _ = B.gbdt_grow_tree_depthwise(p.packed, n_rows, n_features, n_bins, p.grad, p.hess, 4, 1.0,
                                                     1e-3)
    order = order.cpu().numpy()
    assert np.array_equal(np.sort(order), np.arange(n_rows))
    bins = p.bins_cpu.numpy()
    rows_of = {0: np.arange(n_rows)}
    for k, nd in enumerate(nodes):
        rows = rows_of[k]
        assert nd["count"] == rows.size
        if nd["left"] >= 0:
            left = bins[rows, nd["feature"]] <= nd["bin"]
            rows_of[int(nd["left"])], rows_of[int(nd["right"])] = rows[left], rows[~left]
        else:
            at = int(nd["row_begin"])
            assert np.array_equal(order[at:at + rows.size], rows)
