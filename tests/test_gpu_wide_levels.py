"""gbdt_grow_tree_depthwise on levels around the 512 splits up to which the split search forms the siblings: trees of depth
12 whose every split is known beforehand."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_bins,values", [(2, (0, 1)), (60, (7, 41)), (255, (9, 200))])
@pytest.mark.parametrize("deep", [512, 513])
def test_levels_of_more_than_512_splits(deep, n_bins, values):
    """12 two-valued features, five rows for each of their 4,096 combinations, and a gradient that is the sum of
    +-2^-d over the features d.  The levels above depth 10 split everywhere, on feature d (512 splits at depth 9); below,
    the gradients of all but the last `deep` nodes are constant, so that depth 10 has `deep` splits and depth 11
    twice as many.  All sums are exact: nodes, sums and rows have to agree with the rule.  (Without lambda a split gains
    10 x (2^-11)^2 / 0.25 = 9.5e-6 at least, and one of a constant gradient only its rounding, below 1e-6.)"""
    print(f"wide levels, {deep} splits at depth 10, {n_bins} bins", flush=True)
    depth, reps = 12, 5
    combo = np.random.default_rng(deep).permutation(np.repeat(np.arange(1 << depth), reps))
    bit = np.stack([(combo >> (depth - 1 - d)) & 1 for d in range(depth)], axis=1)
    scale = np.array([2.0 ** -d for d in range(depth)])
    contrib = (2 * bit - 1) * scale
    contrib[(combo >> 2) < 1024 - deep, 10:] = 0.0
    grad = contrib.sum(axis=1).astype(np.float32)
    hess = np.full(combo.size, 0.25, np.float32)
    bins = np.where(bit == 1, values[1], values[0]).astype(np.uint8)
    n = combo.size
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).to(DEV), n_bins)
    nodes, order, _ = B.gbdt_grow_tree_depthwise(packed, n, depth, n_bins, torch.from_numpy(grad).to(DEV),
                                                 torch.from_numpy(hess).to(DEV), depth, 0.0, 1e-3, 1e-6)
    order = order.cpu().numpy()
    assert len(nodes) == 2 * 1024 - 1 + 2 * deep + 4 * deep
    level = {0: (0, np.arange(n))}
    splits_at = [0] * (depth + 1)
    for k, nd in enumerate(nodes):
        d, rows = level[k]
        assert nd["count"] == rows.size
        assert nd["sum_grad"] == grad[rows].sum(dtype=np.float64) and nd["sum_hess"] == 0.25 * rows.size
        got_rows = order[nd["row_begin"]:nd["row_begin"] + rows.size]
        if nd["left"] < 0:
            assert np.array_equal(got_rows, rows)
            continue
        assert np.array_equal(np.sort(got_rows), rows)
        splits_at[d] += 1
        assert nd["feature"] == d and nd["bin"] == values[0], (k, d)
        left = bit[rows, d] == 0
        level[int(nd["left"])], level[int(nd["right"])] = (d + 1, rows[left]), (d + 1, rows[~left])
    assert splits_at == [1 << d for d in range(10)] + [deep, 2 * deep, 0]
