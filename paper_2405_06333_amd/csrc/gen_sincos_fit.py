"""Generate sincos_fit.h: polynomial approximations of sin and cos for the
FP64 kernels' sine and cosine on revolutions.

With t = 2 pi f the reduced angle,
  sin t = t + t^3 S(t^2)   and   cos t = 1 - t^2/2 + t^4 C(t^2),
where S and C are Chebyshev interpolants (near-minimax) of
  S(u) = (sin sqrt(u) - sqrt(u)) / u^(3/2),  C(u) = (cos sqrt(u) - 1 + u/2) / u^2
on u in [0, T^2], T = pi/4, after a quarter-turn reduction.  The sine alone
takes a half-turn reduction of the angle in revolutions,
  sin 2 pi f = f H(f^2),   |f| <= 1/4,
H the Chebyshev interpolant in f^2.  The functions are
evaluated with mpmath at 50 digits; the script checks each polynomial,
evaluated in double precision by Horner's rule, against mpmath on a dense
grid and writes the maximum absolute errors into the header.

The structure-factor pass takes both from a table: with the angle in
revolutions reduced to the nearest of 128 parts, f = r - m / 128,
  sin 2 pi f = f A(f^2)   and   cos 2 pi f = 1 + f^2 B(f^2),   |f| <= 1/256,
A and B Chebyshev interpolants in f^2, rotated by the tabulated angle m / 128.

Run: python gen_sincos_fit.py  (writes sincos_fit.h next to this file)
"""
import os

import mpmath as mp
import numpy as np

mp.mp.dps = 50
TERMS_SIN_Q = 6    # t^3 .. t^13
TERMS_COS_Q = 6    # t^4 .. t^14
TERMS_SIN_H = 9    # f .. f^17
PARTS = 128        # table entries per revolution
TERMS_SIN_T = 4    # f .. f^7
TERMS_COS_T = 3    # f^2 .. f^6


def S(u):
    if u == 0:
        return mp.mpf(-1) / 6
    s = mp.sqrt(u)
    return (mp.sin(s) - s) / (u * s)


def C(u):
    if u == 0:
        return mp.mpf(1) / 24
    s = mp.sqrt(u)
    return (mp.cos(s) - 1 + u / 2) / (u * u)


def A(u):
    f = mp.sqrt(u)
    return 2 * mp.pi if u == 0 else mp.sin(2 * mp.pi * f) / f


def B(u):
    f = mp.sqrt(u)
    return -2 * mp.pi ** 2 if u == 0 else (mp.cos(2 * mp.pi * f) - 1) / u


def fit(f, T, terms):
    c = mp.chebyfit(f, [0, T * T], terms)
    return [float(x) for x in c[::-1]]   # ascending powers of u


def horner(c, u):
    p = c[-1]
    for k in range(len(c) - 2, -1, -1):
        p = p * u + c[k]
    return p


def check(c, T, kind):
    t = np.linspace(-float(T), float(T), 40001)
    u = t * t
    if kind == "half":
        got = t * horner(c, u)
        ref = np.array([float(mp.sin(2 * mp.pi * mp.mpf(x))) for x in t])
    elif kind == "sin":
        got = t + t * u * horner(c, u)
        ref = np.array([float(mp.sin(mp.mpf(x))) for x in t])
    else:
        got = 1.0 + u * (-0.5 + u * horner(c, u))
        ref = np.array([float(mp.cos(mp.mpf(x))) for x in t])
    return float(np.max(np.abs(got - ref)))


def check_table(a, b, table):
    r = np.random.default_rng(0).uniform(-4.0, 4.0, 40001)
    m = np.rint(PARTS * r)
    f = r - m / PARTS
    u = f * f
    s, c = f * horner(a, u), 1.0 + u * horner(b, u)
    S, C = table[m.astype(int) % PARTS].T
    sn, cn = C * s + S * c, C * c - S * s
    es = max(abs(g - mp.sin(2 * mp.pi * mp.mpf(x))) for g, x in zip(sn, r))
    ec = max(abs(g - mp.cos(2 * mp.pi * mp.mpf(x))) for g, x in zip(cn, r))
    return float(max(es, ec))


def main():
    q, h = mp.pi / 4, mp.mpf(1) / 4
    sq, cq, sh = fit(S, q, TERMS_SIN_Q), fit(C, q, TERMS_COS_Q), fit(A, h, TERMS_SIN_H)
    es, ec, eh = check(sq, q, "sin"), check(cq, q, "cos"), check(sh, h, "half")
    at, bt = fit(A, mp.mpf(1) / (2 * PARTS), TERMS_SIN_T), fit(B, mp.mpf(1) / (2 * PARTS), TERMS_COS_T)
    table = np.array([[float(mp.sin(2 * mp.pi * m / PARTS)), float(mp.cos(2 * mp.pi * m / PARTS))]
                      for m in range(PARTS)])
    et = check_table(at, bt, table)
    here = os.path.dirname(os.path.abspath(__file__))
    with open(os.path.join(here, "sincos_fit.h"), "w") as f:
        f.write("/* Generated by gen_sincos_fit.py -- do not edit.\n")
        f.write(" * sin t = t + t^3 S(t^2), cos t = 1 - t^2/2 + t^4 C(t^2): Chebyshev interpolants\n")
        f.write(" * of S and C in u = t^2, coefficients in ascending powers of u.  Maximum\n")
        f.write(f" * absolute error in double precision: {es:.2e} (sin, |t| <= pi/4),\n")
        f.write(f" * {ec:.2e} (cos, |t| <= pi/4), {eh:.2e} (sin 2 pi f = f H(f^2), |f| <= 1/4).\n")
        f.write(f" * From the table, sin and cos of 2 pi r: {et:.2e}.\n */\n")
        f.write("#pragma once\n\nnamespace rbe2d {\n\n")
        for name, c, what in (("kSinQuarter", sq, "sin, |t| <= pi/4"), ("kCosQuarter", cq, "cos, |t| <= pi/4"),
                              ("kSinHalf", sh, "sin 2 pi f = f H(f^2), |f| <= 1/4")):
            f.write(f"// {what}\n")
            f.write(f"constexpr int {name}Terms = {len(c)};\n")
            f.write(f"constexpr double {name}[{name}Terms] = {{\n")
            for x in c:
                f.write(f"    {x!r},\n")
            f.write("};\n\n")
        f.write("// from the table: sin 2 pi f = f A(f^2), cos 2 pi f = 1 + f^2 B(f^2), |f| <= 1/256\n")
        f.write(f"constexpr int kParts = {PARTS};\n")
        for name, c in (("kSinPart", at), ("kCosPart", bt)):
            f.write(f"constexpr int {name}Terms = {len(c)};\n")
            f.write(f"constexpr double {name}[{name}Terms] = {{\n")
            for x in c:
                f.write(f"    {x!r},\n")
            f.write("};\n")
        f.write("// sin and cos of 2 pi m / 128\n")
        f.write("static __device__ const double kPartTable[kParts][2] = {\n")
        for s, c in table.tolist():
            f.write(f"    {{{s!r}, {c!r}}},\n")
        f.write("};\n\n}  // namespace rbe2d\n")
    print("max abs errors: sin quarter", es, "cos quarter", ec, "sin half", eh, "table", et)


if __name__ == "__main__":
    main()
