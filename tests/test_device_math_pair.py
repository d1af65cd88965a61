"""The pair (erf S, exp(-S^2)) of the split fluxes (paper_2406_07441_amd/csrc/
lskum_math.h): the polynomials of lskum_math_coef.h evaluated step by step as
the kernels do, each fused multiply-add rounded once, against mpmath's 50-digit
values.

Bounds: a Horner form in fused steps whose last step adds the largest term is
within one unit in the last place plus the fit error; scaling by a constant
adds one rounding (0.5) and the constant's own (0.5), the product S P another
0.5, and beyond |S| = 1 the exponential enters erf through a term of at most
0.16: three units in the last place hold all of them."""
import math
import os
import re
from fractions import Fraction

import numpy as np
import pytest

mp = pytest.importorskip("mpmath")
mp.mp.dps = 50

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2406_07441_amd", "csrc")
ULPS = 3.0


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


@pytest.fixture(scope="module")
def c():
    text = open(os.path.join(CSRC, "lskum_math_coef.h")).read()
    out = {n: [float.fromhex(v.strip()) for v in body.split(",")]
           for n, body in re.findall(r"constexpr double (\w+)\[\d+\] = \{([^}]*)\}", text)}
    out.update({n: float.fromhex(v.strip())
                for n, v in re.findall(r"constexpr double (\w+) = ([^;]+);", text)})
    return out


def horner(coef, x):
    p = coef[0]
    for a in coef[1:]:
        p = fma(p, x, a)
    return p


def exp_lead(x, c):
    k = float(np.rint(x * c["kLog2e"]))
    u = fma(k, c["kLn2Lo"], fma(k, c["kLn2Hi"], -x))
    return math.ldexp(horner(c["kExpN"], u), int(k))


def unit(S, c):
    t = S * S
    return S * horner(c["kErfP"], t), c["kExpHalf"] * horner(c["kExpN"], t - 0.5)


def outer(S, c):
    # the kernels' reciprocal is refined to within a unit in the last place
    x = min(abs(S), 6.0)
    v = (x - 3.0) * (1.0 / (x + 3.0))
    g = exp_lead(-(S * S), c)
    return math.copysign(fma(-g, horner(c["kErfcxW"], v), 1.0), S), g


def worst(pairs):
    return max(abs(got - ref) / math.ulp(ref) if ref else abs(got) for got, ref in pairs)


def test_unit_pair(c):
    rng = np.random.default_rng(2)
    xs = np.concatenate([rng.uniform(-1, 1, 3000), [0.0, 1e-200, -1e-8, 0.5, 0.70710678, -0.9999999]])
    erfs, exps = [], []
    for S in map(float, xs):
        er, g = unit(S, c)
        erfs.append((er, float(mp.erf(mp.mpf(S)))))
        exps.append((g, float(mp.exp(-mp.mpf(S * S)))))
    assert worst(erfs) <= ULPS and worst(exps) <= ULPS


def test_outer_pair(c):
    rng = np.random.default_rng(3)
    xs = np.concatenate([rng.uniform(1, 3, 2000), -rng.uniform(1, 7, 1000), [1.0, -1.0, 5.9999, 6.0, 6.5, 12.0]])
    erfs, exps = [], []
    for S in map(float, xs):
        er, g = outer(S, c)
        erfs.append((er, float(mp.erf(mp.mpf(S)))))
        exps.append((g, float(mp.exp(-mp.mpf(S * S)))))
    assert worst(erfs) <= ULPS and worst(exps) <= ULPS


def test_reduced_exp(c):
    rng = np.random.default_rng(4)
    xs = np.concatenate([rng.uniform(-0.35, 0.35, 1500), rng.uniform(-40, 5, 1500), rng.uniform(-700, 700, 500)])
    assert worst([(exp_lead(float(x), c), float(mp.exp(mp.mpf(float(x))))) for x in xs]) <= ULPS
