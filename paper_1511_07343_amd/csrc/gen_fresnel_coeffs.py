#!/usr/bin/env python3
"""Write fresnel_coeffs.hpp: the polynomial data of the device Fresnel
integrals F(x) = C(x) + i S(x), C(x) = int_0^x cos(pi t^2 / 2) dt.

|x| < 1: the power series C(x) = x sum_n c_n x^(4n), S(x) = x^3 sum_n s_n x^(4n),
  c_n = (-1)^n (pi/2)^(2n) / ((2n)! (4n + 1)),
  s_n = (-1)^n (pi/2)^(2n+1) / ((2n + 1)! (4n + 3)),
  13 terms (the last below 2e-21 at |x| = 1).
x >= 0: the auxiliary functions f, g of F(x) = (1 + i)/2 - (g + i f) exp(i pi x^2 / 2),
  smooth on [0, inf), as polynomials of a variable t in [-1, 1] (Chebyshev fits
  at 40 digits, written out in powers of t):
  x < 3: of f and g themselves in t = 2 x / 3 - 1;
  x >= 3: of phi_f = pi x f and phi_g = pi^2 x^3 g (both -> 1 as x -> inf) in
  t = 18 / x^2 - 1.

Run: python gen_fresnel_coeffs.py  (needs mpmath; the output is committed).
"""
import os

import mpmath as mp

mp.mp.dps = 40

SPLIT = 3  # x at which the two fits meet: few bins of a response lie below it
SMALL_DEGREE, TAIL_DEGREE = 28, 14  # fits within 1e-15 of the 40-digit values (checked below)
SERIES_TERMS = 13


def fg(x):
    x = mp.mpf(x)
    S, C = mp.fresnels(x), mp.fresnelc(x)
    s, c = mp.sin(mp.pi * x * x / 2), mp.cos(mp.pi * x * x / 2)
    # C = 1/2 + f sin - g cos,  S = 1/2 - f cos - g sin
    f = (C - mp.mpf(1) / 2) * s - (S - mp.mpf(1) / 2) * c
    g = -(C - mp.mpf(1) / 2) * c - (S - mp.mpf(1) / 2) * s
    return f, g


def tail(t):
    u = (mp.mpf(t) + 1) / (2 * SPLIT ** 2)
    if u == 0:
        return mp.mpf(1), mp.mpf(1)
    x = 1 / mp.sqrt(u)
    f, g = fg(x)
    return mp.pi * x * f, mp.pi ** 2 * x ** 3 * g


def small(t):
    return fg((mp.mpf(t) + 1) * SPLIT / 2)


def powers(fun, deg):
    """Coefficients in powers of t of the Chebyshev fits of fun's two values."""
    n = deg + 1
    th = [mp.pi * (k + mp.mpf(1) / 2) / n for k in range(n)]
    vals = [fun(mp.cos(t)) for t in th]
    out = []
    for which in (0, 1):
        total = [mp.mpf(0)] * n
        prev, cur = [mp.mpf(1)] + [mp.mpf(0)] * deg, [mp.mpf(0), mp.mpf(1)] + [mp.mpf(0)] * (deg - 1)
        for j in range(n):  # prev holds T_j, cur T_(j+1)
            c = 2 * mp.fsum(v[which] * mp.cos(j * t) for v, t in zip(vals, th)) / n
            c = c / 2 if j == 0 else c
            total = [a + c * b for a, b in zip(total, prev)]
            prev, cur = cur, [2 * a - b for a, b in zip([mp.mpf(0)] + cur[:-1], prev)]
        out.append([float(v) for v in total])
    return out


def horner(cs, t):
    r = cs[-1]
    for c in reversed(cs[:-1]):
        r = r * t + c
    return r


def main():
    here = os.path.dirname(os.path.abspath(__file__))
    series_c = [float((-1) ** n * (mp.pi / 2) ** (2 * n) / (mp.factorial(2 * n) * (4 * n + 1)))
                for n in range(SERIES_TERMS)]
    series_s = [float((-1) ** n * (mp.pi / 2) ** (2 * n + 1) / (mp.factorial(2 * n + 1) * (4 * n + 3)))
                for n in range(SERIES_TERMS)]
    fits = [("Small", small, powers(small, SMALL_DEGREE)), ("Tail", tail, powers(tail, TAIL_DEGREE))]
    worst = 0.0
    for _, fun, coeffs in fits:
        for i in range(0, 200):
            t = -1 + 2 * (i + 0.37) / 200
            for c, e in zip(coeffs, fun(t)):
                worst = max(worst, abs(horner(c, t) - float(e)))
    assert worst < 1e-15, worst
    lines = ["// Generated by gen_fresnel_coeffs.py: polynomial data of the device Fresnel",
             "// integrals (power series below 1; polynomials of the auxiliary functions",
             f"// everywhere, max error in FP64 {worst:.1e} of values up to 1).  Do not edit.",
             "#pragma once", "", "#include <hip/hip_runtime.h>", "", "namespace fdas {",
             "namespace fresnel_data {", ""]
    fmt = lambda v: repr(float(v))  # noqa: E731  (round-trip exact)
    # coefficient arrays live in constant memory: read with uniform indices
    # they become scalar loads, of both functions' coefficients together
    lines.append(f"constexpr double kSplit = {SPLIT}.0;")
    for name, first, second in ([("Series", series_c, series_s)] +
                                [(name, cf, cg) for name, _, (cf, cg) in fits]):
        lines.append(f"__constant__ double k{name}[{len(first)}][2] = {{" +
                     ", ".join(f"{{{fmt(a)}, {fmt(b)}}}" for a, b in zip(first, second)) + "};")
    lines += ["", "}  // namespace fresnel_data", "}  // namespace fdas", ""]
    with open(os.path.join(here, "fresnel_coeffs.hpp"), "w") as f:
        f.write("\n".join(lines))
    print("max error", worst)


if __name__ == "__main__":
    main()
