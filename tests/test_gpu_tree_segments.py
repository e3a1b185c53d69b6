"""Both growers on matrices of several feature tiles, where the gradients and hessians of a round's or level's smaller
children are gathered by segments of the row buffers: trees replayed with the CPU oracle, with the row order written to an
address that is a multiple of 4 bytes and no more, for trees that stop at the last level, before it, and at once."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B

from gpu_util import GpuProblem
from test_gpu_tree import _check_structure, _planted, _replay, _replay_depthwise

pytestmark = pytest.mark.gpu


def _grow(p, n, F, nb, grower, limit, min_gain):
    lib = B.load()
    size = getattr(lib, f"{grower}_scratch_bytes")(n, F, nb, limit)
    scratch = torch.empty(size, dtype=torch.uint8, device="cuda:0")
    nodes = np.zeros(2 * limit - 1 if grower == "gbdt_grow_tree" else (2 << limit) - 1, dtype=B.NODE_DTYPE)
    order = torch.full((n + 2,), -7, dtype=torch.int32, device="cuda:0")
    n_nodes = ctypes.c_int32(0)
    B._check(getattr(lib, grower)(p.packed.data_ptr(), n, F, nb, p.grad.data_ptr(), p.hess.data_ptr(), limit, 1.0, 1e-3,
                                 min_gain, scratch.data_ptr(), size, nodes.ctypes.data, ctypes.byref(n_nodes),
                                 order.data_ptr() + 4, int(torch.cuda.current_stream().cuda_stream)), grower)
    torch.cuda.synchronize()
    order = order.cpu().numpy()
    assert order[0] == -7 and order[n + 1] == -7
    return nodes[:n_nodes.value], order[1:n + 1]


@pytest.mark.parametrize("grower,limit", [("gbdt_grow_tree", 31), ("gbdt_grow_tree", 2),
                                          ("gbdt_grow_tree_depthwise", 5), ("gbdt_grow_tree_depthwise", 1),
                                          ("gbdt_grow_tree_depthwise", 12)])
@pytest.mark.parametrize("n,F,nb", [(20_001, 257, 64), (30_003, 130, 16), (16_385, 120, 255)])
def test_gathered_by_segments(n, F, nb, grower, limit):
    if limit == 12 and F != 130:
        pytest.skip("a tree that stops before its last level is the same step for every tile")
    print(f"{grower} {n}x{F} bins={nb} limit={limit}", flush=True)
    bins, grad, hess = _planted(n, F, nb, n + F)
    p = GpuProblem(bins, nb, grad, hess)
    # (limit 12: far more levels than splits that gain this much, so the rows are not where the last level would leave them)
    min_gain = 60.0 if limit == 12 else 0.0
    nodes, order = _grow(p, n, F, nb, grower, limit, min_gain)
    assert len(nodes) > 1
    _check_structure(nodes, order, bins)
    if grower == "gbdt_grow_tree":
        _replay(nodes, bins, nb, grad, hess, 1.0, 1e-3, min_gain)
    else:
        _replay_depthwise(nodes, bins, nb, grad, hess, 1.0, 1e-3, limit, min_gain)
    nodes, order = _grow(p, n, F, nb, grower, limit, 1e30)      # never split: the rows in their own order
    assert len(nodes) == 1 and np.array_equal(order, np.arange(n))
