"""Wide cells of 256 bins that take two epochs before they are drained, on the CPU, by the functions that the kernel uses: what
the second epoch adds at the first one's scale, where one row may hold all of its sum.

A value is rounded once, by half a unit of its own epoch's scale at most, which is 2^-e, or 2^-(e - 1) where the second epoch's
exponent is one less; the sum of both epochs has to fit the 54-bit field."""
from fractions import Fraction

import numpy as np
import pytest

from paper_1706_08359_amd import binding as B


def exact(values):
    return sum((Fraction(float(v)) for v in values), Fraction(0))


def check(first, second):
    """Returns the difference of the two exponents, 2 where the epochs do not share cells."""
    apart, e, total, added, count = B.gbdt_debug_wide_pair(first, second)
    n = len(first)
    assert count == n
    unit = Fraction(2) ** -e
    if apart == 2:
        assert added == 0 and abs(total * unit - exact(first)) <= n * unit / 2
        return apart
    assert abs(added * unit - exact(second)) <= n * unit * (2 if apart == -1 else 1) / 2, (apart, added)
    assert abs((total - added) * unit - exact(first)) <= n * unit / 2
    assert abs(total) < 2 ** 53
    return apart


def lone(value, n=3, at=1):
    v = np.zeros(n, np.float32)
    v[at] = value
    return v


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("first_sign", [1.0, -1.0])
def test_a_lone_row_holds_its_epochs_sum(sign, first_sign):
    """Sums just around the powers of two at which the exponent steps, and ratios up to nearly four."""
    step = 1.0 / 1.001953125
    seen = set()
    for scale in (1.0, 2.0 ** 20, 2.0 ** -30, 2.0 ** 100):
        for a in (1.0, 1.5, 0.51, step, step * (1 - 2 ** -20), step * (1 + 2 ** -20), 1.99 * step):
            for r in (0.26, 0.5, 0.51, 0.99, 1.0, 1.01, 1.4, 1.5, 1.99, 2.0, 2.01, 3.0, 3.9, 3.99):
                seen.add(check(lone(first_sign * a * scale), lone(sign * a * r * scale)))
    assert seen >= {-1, 0, 1, 2}


def test_figures_by_hand():
    """1.5, then 3: the second epoch's exponent is one less, and 3 at the first one's scale, 2^50, is past 2^51."""
    for v in (3.0, -3.0):
        apart, e, total, added, _ = B.gbdt_debug_wide_pair(lone(1.5), lone(v))
        assert (apart, e) == (-1, 50) and added == int(v) << 50 and total == (3 << 49) + (int(v) << 50)


@pytest.mark.parametrize("draw", ["cauchy", "lognormal", "sparse", "normal"])
def test_heavy_tails(draw):
    rng = np.random.default_rng(5)
    seen = set()
    for _ in range(400):
        pair = []
        for _ in range(2):
            if draw == "cauchy":
                v = rng.standard_cauchy(512)
            elif draw == "lognormal":
                v = rng.lognormal(sigma=2.5, size=512) * rng.choice([-1.0, 1.0], size=512)
            elif draw == "sparse":
                v = rng.normal(size=512) * (rng.random(512) < 1 / 300)
            else:
                v = rng.normal(size=512) * rng.uniform(0.5, 2.0)
            pair.append(v.astype(np.float32))
        seen.add(check(*pair))
    assert seen >= {-1, 0, 1}


def test_all_rows_at_the_largest_value_of_a_pair():
    """Both epochs as large as their exponents allow, all rows of one sign: the field's bound."""
    for n in (1, 2, 511, 512):
        first = np.full(n, 1.99 / 1.001953125 / n, np.float32)
        assert check(first, first * np.float32(2)) == -1
        assert check(-first, -first * np.float32(2)) == -1


def test_zeros_and_the_smallest_and_largest():
    tiny, big = np.float32(2.0 ** -126), np.float32(3e38)
    z = np.zeros(4, np.float32)
    assert check(z, z) == 0
    assert check(z, lone(2.0 ** 26, 4)) == -1 and check(z, lone(-1.9 * 2.0 ** 26, 4)) == -1
    assert check(lone(2.0 ** 26, 4), z) == 1
    assert check(lone(tiny, 4), lone(2 * tiny, 4)) == 0
    # past the largest number an epoch has its cells for itself, and so has the one before it if it comes near
    assert check(np.full(4, 2.0 ** 120, np.float32), lone(big, 4)) == 2
    assert B.gbdt_debug_wide_pair(lone(big, 4), np.full(4, big, np.float32))[0] == 2
    assert B.gbdt_debug_wide_pair(np.full(4, big, np.float32), np.full(4, big, np.float32))[0] == 2


def test_bad_arguments():
    v = np.zeros(513, np.float32)
    with pytest.raises(B.GbdtError):
        B.gbdt_debug_wide_pair(v, v)
    with pytest.raises(B.GbdtError):
        B.gbdt_debug_wide_pair(v[:0], v[:0])
    with pytest.raises(B.GbdtError):
        B.gbdt_debug_wide_pair(v[:3], v[:4])
