"""Blocks of a build whose main tiles are built in halves (wide accumulation, 256 bins): every (tile, half, workgroup) is
one block's, both halves of a (tile, workgroup) are 8 blocks apart, on one XCD, except in the last few, and the remainder
tile, which has no halves, comes last."""
import pytest

from paper_1706_08359_amd import binding as B


@pytest.mark.parametrize("n_features", [1, 16, 17, 32, 33, 64, 70, 96, 100, 137, 500])
@pytest.mark.parametrize("by_column", [False, True])
def test_half_blocks(n_features, by_column):
    g = B.gbdt_debug_geometry(n_features, 256, 1)
    for n_rows in (1000, 9001, 2 ** 25):
        for cols in (1, 3, 8, 9, 56, 170):
            blocks = B.gbdt_debug_half_blocks(n_features, n_rows, cols, by_column).tolist()
            at = {tuple(b): i for i, b in enumerate(blocks)}
            want = {(t, h, c) for t in range(g["n_main"]) for h in (0, 1) for c in range(cols)}
            rest = {(g["n_main"], 0, c) for c in range(cols)} if g["wr"] else set()
            assert set(at) == want | rest and len(blocks) == len(want | rest)
            apart = [at[t, 1, c] - at[t, 0, c] for t in range(g["n_main"]) for c in range(cols)]
            assert sum(d != 8 for d in apart) <= 7
            if rest and want:
                assert min(at[b] for b in rest) > max(at[b] for b in want)
