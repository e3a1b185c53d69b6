"""gbdt_grow_tree on a matrix whose scratch has room for (gradient, hessian) pairs: with a buffer that leaves
out that room (the size that served before it was added) the same tree comes out, a byte less than
that is refused, and the row order is every leaf's rows in ascending order, leaf after leaf."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_tree_with_and_without_room_for_pairs():
    n, F, nb, leaves = 1_100_003, 6, 64, 40
    print(f"tree {n} x {F}", flush=True)
    rng = np.random.default_rng(3)
    bins = rng.integers(0, nb, size=(n, F)).astype(np.uint8)
    grad = np.where((bins[:, 1] > 30) ^ (bins[:, 4] > 40) ^ (rng.random(n) < 0.2), 0.5, -0.5).astype(np.float32)
    hess = np.full(n, 0.25, np.float32)
    packed = B.gbdt_bins_pack(torch.from_numpy(bins).to(DEV), nb)
    g, h = torch.from_numpy(grad).to(DEV), torch.from_numpy(hess).to(DEV)
    nodes, order, _ = B.gbdt_grow_tree(packed, n, F, nb, g, h, leaves, 1.0, 1e-3)
    order = order.cpu().numpy()
    leaf_nodes = sorted((nd for nd in nodes if nd["left"] < 0), key=lambda nd: nd["row_begin"])
    assert len(leaf_nodes) == leaves
    at = 0
    for nd in leaf_nodes:                          # (every leaf: its own rows, each once, ascending)
        rows = order[nd["row_begin"]:nd["row_begin"] + nd["count"]]
        assert nd["row_begin"] == at and (np.diff(rows) > 0).all()
        assert grad[rows].sum(dtype=np.float64) == nd["sum_grad"]
        at += int(nd["count"])
    assert at == n and np.array_equal(np.sort(order), np.arange(n))
    need = B.gbdt_grow_tree_scratch_bytes(n, F, nb, leaves)
    least = need - (8 * n + 255) // 256 * 256
    scratch = torch.empty(need, dtype=torch.uint8, device=DEV)
    for size, ok in ((least, True), (least - 1, False)):
        nodes2 = np.zeros(2 * leaves - 1, dtype=B.NODE_DTYPE)
        order2 = torch.empty(n, dtype=torch.int32, device=DEV)
        n_nodes = ctypes.c_int32(0)
        rc = B.load().gbdt_grow_tree(packed.data_ptr(), n, F, nb, g.data_ptr(), h.data_ptr(), leaves, 1.0, 1e-3, 0.0,
                                     scratch.data_ptr(), size, nodes2.ctypes.data, ctypes.byref(n_nodes),
                                     order2.data_ptr(), int(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert (rc == 0) == ok
        if ok:
            assert n_nodes.value == len(nodes) and np.array_equal(nodes2[:n_nodes.value], nodes)
            assert np.array_equal(order2.cpu().numpy(), order)
