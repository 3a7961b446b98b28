"""Generate exp2_fit.h: the polynomial of the FP64 pair kernel's exponential.

2^f = 1 + f E(f) for |f| <= 1/2, where E is the Chebyshev interpolant
(near-minimax) of (2^f - 1) / f.  The function is evaluated with mpmath at 50
digits; the script checks 1 + f E(f), evaluated in double precision by
Horner's rule, against mpmath on a dense grid and writes the maximum relative
error into the header.

Run: python gen_exp2_fit.py  (writes exp2_fit.h next to this file)
"""
import os

import mpmath as mp
import numpy as np

mp.mp.dps = 50
TERMS = 11


def E(f):
    return mp.log(2) if f == 0 else mp.expm1(f * mp.log(2)) / f


def main():
    c = [float(x) for x in mp.chebyfit(E, [mp.mpf(-1) / 2, mp.mpf(1) / 2], TERMS)[::-1]]
    f = np.linspace(-0.5, 0.5, 40001)
    p = np.full_like(f, c[-1])
    for k in range(TERMS - 2, -1, -1):
        p = p * f + c[k]
    got = 1.0 + f * p
    err = float(max(abs(mp.mpf(g) / mp.power(2, mp.mpf(x)) - 1) for g, x in zip(got[::8], f[::8])))
    here = os.path.dirname(os.path.abspath(__file__))
    with open(os.path.join(here, "exp2_fit.h"), "w") as out:
        out.write("/* Generated by gen_exp2_fit.py -- do not edit.\n")
        out.write(" * 2^f = 1 + f E(f), |f| <= 1/2: Chebyshev interpolant of E, ascending powers of f.\n")
        out.write(f" * Maximum relative error in double precision: {err:.2e}.\n */\n")
        out.write("#pragma once\n\nnamespace rbe2d {\n\n")
        out.write(f"constexpr int kExp2Terms = {TERMS};\n")
        out.write("constexpr double kExp2[kExp2Terms] = {\n")
        for x in c:
            out.write(f"    {x!r},\n")
        out.write("};\n\n}  // namespace rbe2d\n")
    print("max relative error", err)


if __name__ == "__main__":
    main()
