"""The constants of the FP64 negative half powers in the kernels' source: with e = 1 - x y^2,
x^(-P/2) = y^P kappa ((e + h)^2 + c), so kappa = P (P + 2) / 8, 2 kappa h = P / 2 and
kappa (h^2 + c) = 1.  The first holds exactly, the last to a quarter of an ulp (a fixed relative
error of every term), the slope to 1e-8 (it multiplies |e| < 1.1e-7: 1e-15 x 1e-7 is nothing,
and 1e-8 x 1e-7 is still ten times below an ulp)."""
import os
import re
from fractions import Fraction as F

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1606_03743_amd", "csrc",
                   "kernels.hip")


def constants(p):
    m = re.search(r"struct HalfPower<%d> \{ static constexpr double kHalf = (\S+), kRest = (\S+), kappa = (\S+); \};" % p,
                  open(SRC).read())
    return float.fromhex(m.group(1)), float.fromhex(m.group(2)), float(m.group(3))


POWERS = [int(p) for p in re.findall(r"struct HalfPower<(\d)> \{", open(SRC).read())]


@pytest.mark.parametrize("p", POWERS)
def test_constants(p):
    half, rest, kappa = constants(p)
    h = F(half) - 1
    assert F(kappa) == F(p * (p + 2), 8)
    assert abs(F(kappa) * (h * h + F(rest)) - 1) <= F(1, 2 ** 54)
    assert abs(2 * F(kappa) * h - F(p, 2)) <= F(1, 10 ** 8)


@pytest.mark.parametrize("p", POWERS)
def test_rounding(p):
    """The sequence of operations, each rounded to FP64 (products and sums in extended precision
    first, as the fused instructions do), from an estimate with the hardware's error (5.2e-8):
    within 5 half-ulp steps (y^2 counts half, one each for y^P's products, the square, the last
    product) of the power."""
    half, rest, kappa = constants(p)
    rng = np.random.default_rng(p)
    n = 100_000
    x = rng.uniform(1.0, 4.0, n) * 4.0 ** rng.integers(-20, 21, n)
    y = (1.0 / np.sqrt(x)) * (1.0 + rng.uniform(-5.2e-8, 5.2e-8, n))
    L = np.longdouble
    y2 = y * y
    t = (L(half) - L(x) * L(y2)).astype(np.float64)
    m = (L(t) * L(t) + L(rest)).astype(np.float64)
    yp = y if p == 1 else y2 * y if p == 3 else (y2 * y2) * y
    got = L(yp * m) * L(kappa)
    want = L(x) ** (L(-p) / 2)
    assert float(np.max(np.abs(got / want - 1))) <= 5 * 2.0 ** -53
