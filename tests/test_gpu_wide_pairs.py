"""Wide sums of 256 bins, whose cells are drained once in two epochs (of 512 rows) when their scales allow it: against the oracle, with
magnitudes that stay, that change a little and that change a lot from epoch to epoch, zeros, one sign, lone rows that hold an
epoch's sum, heavy tails, and sums past fp32 in between; whole tiles and halves, roots, lists and batches, odd and even numbers of epochs.

Where all statistics are small multiples of a power of two every sum is exact and has to agree bit for bit; elsewhere within
2^-23 of the value, the rounding of what is stored, and 1e-12 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

from paper_1706_08359_amd import binding as B
from tests.gpu_util import GpuProblem

pytestmark = pytest.mark.gpu

N_ROWS = 12_345


def stats(kind, rng):
    g = rng.integers(-3, 4, size=N_ROWS) * 0.5
    h = rng.integers(0, 5, size=N_ROWS) * 0.25
    epoch = np.arange(N_ROWS) // 512
    if kind == "one_sign":
        g, h = np.abs(g) + 0.5, -h - 0.25
    elif kind == "a_little":
        g, h = g * 2.0 ** (epoch % 2), h * 2.0 ** (epoch // 2 % 2)
    elif kind == "a_lot":
        g, h = g * 2.0 ** (epoch * 5 % 17), h * 2.0 ** (-(epoch * 3 % 11.0))
    elif kind == "zeros":
        g, h = g * (epoch % 3 > 0), h * (epoch % 4 > 1)
    elif kind == "rounded":
        g, h = rng.normal(size=N_ROWS) * 10.0 ** (epoch % 5 / 5), rng.uniform(0.01, 1.0, size=N_ROWS)
    return g.astype(np.float32), h.astype(np.float32)


def agrees(got_t, p, idx, n_leaf, exact, what):
    got, ref = B.hist_to_numpy(got_t), p.oracle(idx, n_leaf=n_leaf)
    assert np.array_equal(got["count"].astype(np.int64), ref["count"].astype(np.int64)), what
    for k, total in zip(("grad", "hess"), p.leaf_abs_sums(idx, n_leaf)):
        d = np.abs(got[k].astype(np.float64) - ref[k])
        assert (d <= (0.0 if exact else 2.0 ** -23 * np.abs(ref[k]) + 1e-12 * total)).all(), (what, k)


@pytest.mark.parametrize("kind", ["plain", "one_sign", "a_little", "a_lot", "zeros", "rounded"])
# (with 600 and 1,200 features the workgroups of a root of 25 epochs have two and five each, with fewer features one)
@pytest.mark.parametrize("n_features,n_bins", [(28, 255), (10, 256), (40, 200), (70, 255), (600, 255), (1200, 255)])
def test_two_epochs_a_drain(n_features, n_bins, kind):
    print(f"wide pairs {n_features} x {n_bins} {kind}", flush=True)
    rng = np.random.default_rng(n_features)
    bins = rng.integers(0, n_bins, size=(N_ROWS, n_features)).astype(np.uint8)
    bins[:, 0] = 3                                                         # all rows of both epochs in one cell
    grad, hess = stats(kind, rng)
    p = GpuProblem(bins, n_bins, grad, hess)
    exact = kind != "rounded"
    B.gbdt_set_wide_accumulation(True)
    B.gbdt_set_deterministic(True)
    try:
        for n in (N_ROWS, 512, 1024, 1025, 2048, 11 * 512, 12 * 512 + 1):
            agrees(p.build(n_leaf=n), p, None, n, exact, ("root", n))
        lists = [np.sort(rng.choice(N_ROWS, size=n, replace=False)).astype(np.int32) for n in (11_000, 2_000, 1_536, 900)]
        for idx in lists:
            agrees(p.build(idx), p, idx, None, exact, ("list", len(idx)))
        offs = np.concatenate([[0], np.cumsum([len(i) for i in lists])])
        hists = B.gbdt_hist_build_batch(p.packed, N_ROWS, n_features, n_bins,
                                        torch.from_numpy(np.concatenate(lists)).to(p.dev), offs, p.grad, p.hess)
        for k, idx in enumerate(lists):
            agrees(hists[k], p, idx, None, exact, ("batch", len(idx)))
    finally:
        B.gbdt_set_wide_accumulation(False)
        B.gbdt_set_deterministic(False)


def lone_rows(ratio, noise, rng):
    """One row holds (nearly) all of its epoch's sum, in every second epoch `ratio` times that of the epoch before."""
    first = np.array([1.5, 100.0, 0.75, 1.0])[np.arange(N_ROWS) // 1024 % 4]
    v = noise * rng.integers(-1, 2, size=N_ROWS).astype(np.float64)
    at = np.arange(0, N_ROWS - 512, 512) + rng.integers(0, 512, size=N_ROWS // 512)
    v[at] = first[at] * np.where(at // 512 % 2, ratio, 1.0)
    return v.astype(np.float32)


@pytest.mark.parametrize("noise", [0.0, 2.0 ** -11])
@pytest.mark.parametrize("n_features", [28, 70, 600])
def test_a_lone_row_holds_an_epochs_sum(n_features, noise):
    """Every value is a multiple of 2^-11 and every sum below 2^12: exact, also as it is stored."""
    rng = np.random.default_rng(n_features)
    bins = rng.integers(0, 255, size=(N_ROWS, n_features)).astype(np.uint8)
    ratios = [2.0, -2.0, 3.0, -3.5, 1.9375, 0.5, -0.28125, 1.0]
    p = GpuProblem(bins, 255, np.zeros(N_ROWS, np.float32), np.zeros(N_ROWS, np.float32))
    lists = [np.sort(rng.choice(N_ROWS, size=n, replace=False)).astype(np.int32) for n in (11_000, 2_000)]
    lists += [np.arange(a, b, dtype=np.int32) for a, b in ((0, 2048), (2048, 3072), (1024, 5632))]  # whole epochs of the matrix
    offs = np.concatenate([[0], np.cumsum([len(i) for i in lists])])
    flat = torch.from_numpy(np.concatenate(lists)).to(p.dev)
    B.gbdt_set_wide_accumulation(True)
    try:
        for k, r in enumerate(ratios):
            print(f"lone rows {n_features} noise {noise} ratio {r}", flush=True)
            for a, ratio in (("grad", r), ("hess", ratios[(k + 3) % len(ratios)])):
                setattr(p, a + "_cpu", torch.from_numpy(lone_rows(ratio, noise, rng)))
                setattr(p, a, getattr(p, a + "_cpu").to(p.dev))
            for n in (N_ROWS, 1024, 2048, 6 * 512):
                agrees(p.build(n_leaf=n), p, None, n, True, ("root", r, n))
            for idx in lists:
                agrees(p.build(idx), p, idx, None, True, ("list", r, len(idx)))
            hists = B.gbdt_hist_build_batch(p.packed, N_ROWS, n_features, 255, flat, offs, p.grad, p.hess)
            for i, idx in enumerate(lists):
                agrees(hists[i], p, idx, None, True, ("batch", r, len(idx)))
    finally:
        B.gbdt_set_wide_accumulation(False)


@pytest.mark.parametrize("n_features", [28, 600])
def test_heavy_tails(n_features):
    """Cauchy gradients, log-normal hessians: about one pair in a hundred has a row that is past 2^51 at the first epoch's scale."""
    rng = np.random.default_rng(7)
    bins = rng.integers(0, 255, size=(N_ROWS, n_features)).astype(np.uint8)
    lists = [np.sort(rng.choice(N_ROWS, size=2_000, replace=False)).astype(np.int32) for _ in range(200)]
    p = GpuProblem(bins, 255, rng.standard_cauchy(N_ROWS).astype(np.float32), rng.lognormal(sigma=2.5, size=N_ROWS).astype(np.float32))
    past = 0
    for v in (p.grad_cpu.numpy(), p.hess_cpu.numpy()):
        for idx in lists:
            apart, e = B.gbdt_debug_wide_pair(v[idx[:512]], v[idx[512:1024]])[:2]
            past += apart == -1 and np.abs(v[idx[512:1024]]).max() > 2.0 ** (51 - e)
    assert past > 0
    B.gbdt_set_wide_accumulation(True)
    try:
        agrees(p.build(), p, None, None, False, "root")
        hists = B.gbdt_hist_build_batch(p.packed, N_ROWS, n_features, 255, torch.from_numpy(np.concatenate(lists)).to(p.dev),
                                        np.arange(201) * 2_000, p.grad, p.hess)
        for i, idx in enumerate(lists):
            agrees(hists[i], p, idx, None, False, ("batch", i))
    finally:
        B.gbdt_set_wide_accumulation(False)


def test_long_units_of_many_epochs():
    """A root whose workgroups take long units from the run-time hand-out."""
    n_rows, n_features = 60_000, 2000
    rng = np.random.default_rng(3)
    bins = rng.integers(0, 255, size=(n_rows, n_features)).astype(np.uint8)
    g = B.gbdt_debug_geometry(n_features, 255, n_rows)
    grad = (rng.integers(-3, 4, size=n_rows) * 0.5).astype(np.float32)
    hess = (rng.integers(1, 5, size=n_rows) * 0.25).astype(np.float32)
    assert -(-n_rows // 512) > 12 * g["wgs"]
    p = GpuProblem(bins, 255, grad, hess)
    B.gbdt_set_wide_accumulation(True)
    try:
        agrees(p.build(), p, None, None, True, "root")
    finally:
        B.gbdt_set_wide_accumulation(False)


def test_a_sum_past_fp32_between_others():
    n_rows, big = 4 * 512, np.float32(3e38)
    rng = np.random.default_rng(4)
    bins = rng.integers(2, 200, size=(n_rows, 28)).astype(np.uint8)
    grad, hess = np.ones(n_rows, np.float32), np.ones(n_rows, np.float32)
    for e in (1, 2):                                                        # epochs 1 and 2 of four
        rows = np.arange(512 * e, 512 * e + 5)
        bins[rows], grad[rows], hess[rows] = 1, big if e == 1 else -big, big / 16
    p = GpuProblem(bins, 200, grad, hess)
    B.gbdt_set_wide_accumulation(True)
    try:
        got = B.hist_to_numpy(p.build(np.arange(n_rows, dtype=np.int32)))
    finally:
        B.gbdt_set_wide_accumulation(False)
    assert (got["count"][:, 1] == 10).all() and (got["grad"][:, 1] == 0).all()
    assert (np.abs(got["hess"][:, 1].astype(np.float64) - 10 * np.float64(big / 16)) <= 2.0 ** -23 * 2e38).all()
