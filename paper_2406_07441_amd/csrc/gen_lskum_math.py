"""Writes the polynomial coefficients of the solver kernels' exp and erf
(lskum_math_coef.h) from near-minimax Chebyshev fits in 50-digit arithmetic
(mpmath.chebyfit):

  exp: after x = k ln2 + r, |r| <= ln2/2,  e^r = 1 + r + r^2 Q(r),
       Q(r) = (e^r - 1 - r)/r^2 of degree 10 (fit error 1.4e-18);
  erf: for |x| < 1,  erf(x) = x P(x^2),
       P(t) = erf(sqrt t)/sqrt t on [0, 1] of degree 11 (fit error 7.4e-18);
  exp(-t) for 0 <= t < 1 without a range reduction: E(t - 1/2),
       E(u) = e^(-u) on |u| <= 1/2 of degree 12, of which the callers take
       e^(-1/2) (fit error 5.0e-18, of exp(-t) 3.0e-18);
  erf for 1 <= |x|: sign(x) (1 - e^(-x^2) W(v)), v = (|x| - 3)/(|x| + 3),
       W(v) = erfcx(|x|) on 1 <= |x| <= 6 of degree 14 (fit error 1.0e-17).

Coefficients are listed from the highest degree down (Horner order) as C99
hexadecimal floating literals, each the double nearest the fitted value.
Run:  python gen_lskum_math.py > lskum_math_coef.h
"""
import mpmath as mp

mp.mp.dps = 50


def exp_q(r):
    return (mp.exp(r) - 1 - r) / (r * r) if r != 0 else mp.mpf(1) / 2


def erf_p(t):
    return mp.erf(mp.sqrt(t)) / mp.sqrt(t) if t != 0 else 2 / mp.sqrt(mp.pi)


def exp_neg(u):
    return mp.exp(-u)


def erfcx_w(v):
    x = 3 * (1 + v) / (1 - v)
    return mp.exp(x * x) * mp.erfc(x)


def fits():
    half_ln2 = mp.log(2) / 2
    q, eq = mp.chebyfit(exp_q, [-half_ln2, half_ln2], 11, error=True)
    p, ep = mp.chebyfit(erf_p, [0, 1], 12, error=True)
    n, en = mp.chebyfit(exp_neg, [-mp.mpf(1) / 2, mp.mpf(1) / 2], 13, error=True)
    w, ew = mp.chebyfit(erfcx_w, [-mp.mpf(1) / 2, mp.mpf(1) / 3], 15, error=True)
    return (q, eq), (p, ep), (n, en), (w, ew)


def table(name, coef):
    vals = [float(c).hex() for c in coef]
    body = ",\n    ".join(vals)
    return f"constexpr double {name}[{len(vals)}] = {{\n    {body}}};\n"


def main():
    (q, eq), (p, ep), (n, en), (w, ew) = fits()
    ln2 = mp.log(2)
    ln2_hi = float(ln2)
    ln2_lo = float(ln2 - mp.mpf(ln2_hi))
    print("// Generated by gen_lskum_math.py; do not edit.")
    print(f"// Q(r) = (e^r - 1 - r)/r^2 on |r| <= ln2/2, degree 10, fit error {mp.nstr(eq, 3)}")
    print(table("kExpQ", q))
    print(f"// P(t) = erf(sqrt t)/sqrt t on [0, 1], degree 11, fit error {mp.nstr(ep, 3)}")
    print(table("kErfP", p))
    print(f"// E(u) = e^(-u) on [-1/2, 1/2], degree 12, fit error {mp.nstr(en, 3)}")
    print(table("kExpN", n))
    print(f"// W(v) = erfcx(3 (1 + v)/(1 - v)) on [-1/2, 1/3], degree 14, fit error {mp.nstr(ew, 3)}")
    print(table("kErfcxW", w))
    print(f"constexpr double kExpHalf = {float(mp.exp(-mp.mpf(1) / 2)).hex()};")
    print(f"constexpr double kLog2e = {float(1 / ln2).hex()};")
    print(f"constexpr double kLn2Hi = {ln2_hi.hex()};")
    print(f"constexpr double kLn2Lo = {ln2_lo.hex()};")


if __name__ == "__main__":
    main()
