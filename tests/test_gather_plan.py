"""The gather of a batch's statistics by parts of the lists takes several lists a launch and gives their places relative to the
launch's first one in 32 bits: every list starts where the call's offsets say, also where the lists of one launch hold
2^32 entries and more together.  (Lists of one build launch, 224, hold fewer, as gbdt_hist_build_batch requires.)"""
import numpy as np
import pytest

from paper_1706_08359_amd import binding as B


@pytest.mark.parametrize("n_leaves,length", [(1, 7), (300, 5), (301, 5), (700, 0), (225, 19_100_000), (300, 19_100_000),
                                             (450, 19_100_000), (300, 2 ** 32 // 300 + 1), (3, 2 ** 31 - 1)])
@pytest.mark.parametrize("start", [0, 12345])
def test_lists_start_where_the_offsets_say(n_leaves, length, start):
    rng = np.random.default_rng(n_leaves)
    sizes = np.full(n_leaves, length, np.int64) - (rng.integers(0, length // 2000 + 1, size=n_leaves))
    offs = start + np.concatenate([[0], np.cumsum(sizes)])
    launch, position = B.gbdt_debug_gather_plan(offs)
    assert np.array_equal(position, offs[:-1])
    assert launch[0] == 0 and set(np.diff(launch)) <= {0, 1}
    for k in range(launch[-1] + 1):
        mine = np.flatnonzero(launch == k)
        assert len(mine) <= 300 and offs[mine[-1] + 1] - offs[mine[0]] < 2 ** 32
