"""Prints the polynomial of phi_lower in lskum_mlp.hip.

P(a) = log2 Phi(-a) on [0, 6] (Phi the normal distribution function), degree 10,
P(0) = -1, minimax in the error of Phi(-a), which is the error of
gelu(-a) = -a Phi(-a) per unit of a.  The linear programme bounds Phi ln2 |P - log2 Phi|
on 20,001 points; coefficients are listed from the highest degree down, rounded to
fp32, with the error that the rounded ones have.

Run: python3 gen_lskum_gelu.py
"""
import numpy as np
from scipy.optimize import linprog
from scipy.special import log_ndtr, ndtr

DEGREE, END = 10, 6.0


def error(coef, a):
    """Relative to a, of -a 2^P(a) as gelu(-a)."""
    return ndtr(-a) * np.expm1(np.polyval(coef, a) * np.log(2) - log_ndtr(-a))


def fit():
    a = np.linspace(0.0, END, 20001)
    w = 1e6 * np.log(2) * ndtr(-a)
    log2phi = log_ndtr(-a) / np.log(2)
    T = np.polynomial.chebyshev.chebvander(2 * a / END - 1, DEGREE)
    one = np.ones((a.size, 1))
    r = linprog(np.r_[np.zeros(DEGREE + 1), 1.0],
                A_ub=np.r_[np.c_[T * w[:, None], -one], np.c_[-T * w[:, None], -one]],
                b_ub=np.r_[w * log2phi, -w * log2phi],
                A_eq=np.r_[T[0], 0.0][None], b_eq=[-1.0],
                bounds=[(None, None)] * (DEGREE + 1) + [(0, None)], method="highs",
                options=dict(primal_feasibility_tolerance=1e-10,
                             dual_feasibility_tolerance=1e-10))
    p = np.polynomial.chebyshev.Chebyshev(r.x[:-1], domain=[0.0, END])
    return p.convert(kind=np.polynomial.Polynomial).coef[::-1].astype(np.float32)


if __name__ == "__main__":
    c = fit()
    print(f"// error {np.abs(error(c.astype(np.float64), np.linspace(0, END, 100001))).max():.1e}")
    for k, v in enumerate(c):
        print(f"    float p = {v:.9e}f;" if k == 0 else f"    p = fmaf(p, a, {v:.9e}f);")
