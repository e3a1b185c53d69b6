"""Which kernel a leaf's build takes, on the CPU: for short leaves where a tile has one workgroup, and with 256 bins where a workgroup
has one or two epochs; for long ones everywhere else."""
import pytest

from paper_1706_08359_amd import binding as B

N_ROWS = 3_000_000


def plan(n_features, n_bins, n, indexed=False):
    return B.gbdt_debug_leaf_plan(N_ROWS, n_features, n_bins, n, indexed)


@pytest.mark.parametrize("indexed", [False, True])
@pytest.mark.parametrize("n_features,n_bins", [(28, 255), (500, 256), (60, 64), (2000, 63), (40, 16), (700, 9)])
def test_one_workgroup_a_tile_or_few_epochs(n_features, n_bins, indexed):
    seen = set()
    for n in [1, 511, 512, 2048, 2049, 5_000, 20_000, 60_000, 100_000, 300_000, 1_000_000, N_ROWS]:
        p = plan(n_features, n_bins, n, indexed)
        expect = p["one_unit_each"] and (p["wgs"] == 1 or (n_bins > 64 and p["unit_epochs"] <= 2))
        assert p["short"] == expect, (n, p)
        seen.add(p["short"])
        B.gbdt_set_wide_accumulation(True)
        try:
            p = plan(n_features, n_bins, n, indexed)
        finally:
            B.gbdt_set_wide_accumulation(False)
        assert p["short"] == (n_bins > 64 or (p["one_unit_each"] and p["wgs"] == 1)), (n, p)
    assert seen == {0, 1}


def test_lines_of_the_rule():
    """500 features of 256 bins: 32 workgroups a tile fit the machine."""
    for epochs, wgs, short in ((4, 1, 1), (5, 5, 1), (32, 32, 1), (64, 32, 1), (65, 22, 0), (384, 32, 0), (385, 32, 0)):
        p = plan(500, 255, 512 * epochs)
        assert (p["wgs"], p["short"]) == (wgs, short), (epochs, p)
    # 32 tiles of 64 bins: 24 workgroups; more tiles than workgroups that fit: one
    for n_features, epochs, wgs, short in ((2000, 4, 1, 1), (2000, 5, 5, 0), (2000, 24, 24, 0), (50_000, 12, 1, 1), (50_000, 13, 1, 0)):
        p = plan(n_features, 64, 512 * epochs)
        assert (p["wgs"], p["short"]) == (wgs, short), (n_features, epochs, p)
