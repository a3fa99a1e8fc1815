"""Writes sincos_table.h: the first octant of the 4,096-entry phasor table and
the polynomials of the angle left over inside a cell (phasor_table.h).

Entry k of the table is (cos, sin)(2 pi k / 4096), each correctly rounded.
The header holds k = 0 .. 512; the other octants follow by exchanging the two
and changing signs, exactly.

Inside a cell, |d| <= 1/8192 turns, the angle is taken as

    sin(2 pi d) = d (S0 + S1 q),   cos(2 pi d) - 1 = q (C0 + C1 q),   q = d^2,

least-squares fits on Chebyshev nodes of q at 50 digits (absolute error), then
rounded to FP64.

Run:  python gen_sincos_table.py   (rewrites sincos_table.h next to it)
"""
import os

import mpmath as mp

mp.mp.dps = 50
N = 4096
H = mp.mpf(1) / (2 * N)


def _lsq(f, n, weight):
    m, b = 200, H * H
    ts = [b / 2 + b / 2 * mp.cos(mp.pi * (2 * k + 1) / (2 * m)) for k in range(m)]
    A, y = mp.matrix(m, n), mp.matrix(m, 1)
    for i, t in enumerate(ts):
        for k in range(n):
            A[i, k] = weight(t) * t ** k
        y[i] = weight(t) * f(t)
    c = mp.lu_solve(A.T * A, A.T * y)
    return [float(c[k]) for k in range(n)]


def main():
    S = _lsq(lambda t: mp.sin(2 * mp.pi * mp.sqrt(t)) / mp.sqrt(t), 2, mp.sqrt)
    C = _lsq(lambda t: (mp.cos(2 * mp.pi * mp.sqrt(t)) - 1) / t, 2, lambda t: t)
    es = ec = mp.mpf(0)
    for i in range(2001):
        d = H * i / 2000
        q = d * d
        es = max(es, abs(d * (mp.mpf(S[0]) + mp.mpf(S[1]) * q) - mp.sin(2 * mp.pi * d)))
        ec = max(ec, abs(q * (mp.mpf(C[0]) + mp.mpf(C[1]) * q) - (mp.cos(2 * mp.pi * d) - 1)))
    lines = ["// Generated by gen_sincos_table.py; do not edit.",
             "// Max |error| of the rounded polynomials in a cell: "
             f"{mp.nstr(es, 3)} (sin), {mp.nstr(ec, 3)} (cos).",
             "#pragma once", "namespace swv {",
             f"constexpr double kCellS[2] = {{{S[0]!r}, {S[1]!r}}};",
             f"constexpr double kCellC[2] = {{{C[0]!r}, {C[1]!r}}};",
             "// (cos, sin)(2 pi k / 4096), k = 0 .. 512",
             "static __device__ const double kOctant[513][2] = {"]
    for k in range(N // 8 + 1):
        x = 2 * mp.pi * k / N
        lines.append(f"    {{{float(mp.cos(x))!r}, {float(mp.sin(x))!r}}},")
    lines += ["};", "}  // namespace swv"]
    out = os.path.join(os.path.dirname(os.path.abspath(__file__)), "sincos_table.h")
    with open(out, "w") as f:
        f.write("\n".join(lines) + "\n")
    print("wrote", out, "errors", mp.nstr(es, 3), mp.nstr(ec, 3))


if __name__ == "__main__":
    main()
