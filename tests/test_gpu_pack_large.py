"""gbdt_bins_pack on both sides of the size from which its copies are written past the caches (256 MiB): the column copy
and the counts of a build from the tiles, on the device."""
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_features,n_bins", [(131, 255), (130, 64), (257, 13)])
@pytest.mark.parametrize("large", [False, True])
def test_pack_around_the_cache_size(n_features, n_bins, large):
    g = B.gbdt_debug_geometry(n_features, n_bins, 1)
    n = (256 << 20) // (g["row_bytes"] + n_features) + (3001 if large else -3001)
    print(f"pack {n} x {n_features}, {n_bins} bins", flush=True)
    assert (B.gbdt_bins_packed_bytes(n, n_features, n_bins) > 256 << 20) == large
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    bins = torch.randint(0, n_bins, (n, n_features), generator=gen, device="cuda", dtype=torch.uint8)
    packed = B.gbdt_bins_pack(bins, n_bins, fuse=False)
    stride = (n + 255) // 256 * 256
    base = (n * g["row_bytes"] + 512 * 64 + 255) // 256 * 256
    cols = packed[base:base + n_features * stride].reshape(n_features, stride)[:, :n]
    assert torch.equal(cols, bins.t())
    ones = torch.ones(n, device="cuda")
    hist = B.gbdt_hist_build(packed, n, n_features, n_bins, None, n, ones, ones)
    counts = hist.view(torch.int32)[..., 2]
    for f in range(n_features):
        assert torch.equal(counts[f], torch.bincount(bins[:, f].to(torch.int64), minlength=n_bins).to(torch.int32)), f
