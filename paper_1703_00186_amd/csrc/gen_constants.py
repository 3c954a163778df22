"""Generates d2q37_constants.h: the D2Q37 velocity set, weights and Hermite tables.

The GPU kernels take every model constant from this header as a compile-time
literal, so that after full unrolling the coefficients of the collision sit
in scalar registers or instruction operands rather than in memory (the
constant-cache effect the paper measures for its CUDA collide, Sec. 5).

Derivation (Sec. 2: 37 populations that hop at most three sites; Hermite basis):
  * hops e_l: every integer vector with |e|^2 <= 10, ordered by e_x descending
    then e_y ascending (so e_0 = (3,-1), e_1 = (3,0) as the propagate listing
    of Sec. 4, Fig. 4 gathers them, and e_{36-l} = -e_l);
  * lattice velocities c_l = r e_l, with the 8 family weights and r solved
    from sum_l w_l c_lx^p c_ly^q = E[z^p] E[z^q] (standard normal z) for the
    nine even (p, q) of total degree <= 8, plus (4,4); the rule is then exact
    to degree 9.  Solved with mpmath at 50 digits and rounded to double;
  * the powers of r and the even moments of the weights that the coefficient
    form of the state needs (d2q37_coeff.h), each rounded once, the moments
    those of the rounded weights: what the map from moments to coefficients
    takes must be what the populations give back.
Run as a script to rewrite the header; ``check()`` compares a fresh solve
with the header on disk.
"""

from __future__ import annotations

import os
import struct
import sys

import mpmath as mp

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(HERE, "d2q37_constants.h")

FAMILIES = [(0, 0), (0, 1), (1, 1), (0, 2), (1, 2), (2, 2), (0, 3), (1, 3)]
CONDITIONS = [(0, 0), (2, 0), (4, 0), (2, 2), (6, 0), (4, 2), (8, 0), (6, 2), (4, 4)]


def hops():
    return [(ex, ey) for ex in range(3, -4, -1) for ey in range(-3, 4) if ex * ex + ey * ey <= 10]


def family(e):
    a, b = sorted((abs(e[0]), abs(e[1])))
    return FAMILIES.index((a, b))


def solve(dps: int = 50):
    mp.mp.dps = dps
    E = hops()

    def gm(p):
        return mp.mpf(mp.fac2(p - 1)) if p > 0 else mp.mpf(1)

    def residual(*x):
        W, r = x[:8], x[8]
        out = []
        for p, q in CONDITIONS:
            s = mp.mpf(0)
            for e in E:
                s += W[family(e)] * (r * e[0]) ** p * (r * e[1]) ** q
            out.append(s - gm(p) * gm(q))
        return out

    # start from the isotropic guess of a Gaussian sampled at the hops
    r0 = mp.mpf("1.2")
    w0 = [mp.exp(-(r0 * r0) * (a * a + b * b) / 2) for a, b in FAMILIES]
    norm = sum(w0[family(e)] for e in E)
    x0 = [w / norm for w in w0] + [r0]
    sol = mp.findroot(residual, x0)
    W = [sol[i] for i in range(8)]
    r = sol[8]
    if max(abs(v) for v in residual(*W, r)) > mp.mpf(10) ** (-(dps - 10)):
        raise RuntimeError("quadrature solve did not converge")
    if min(W) <= 0:
        raise RuntimeError("non-positive weight")
    return E, W, r


def hermite(n, x):
    return [mp.mpf(1), x, x * x - 1, x ** 3 - 3 * x, x ** 4 - 6 * x * x + 3][n]


def hexf(v) -> str:
    d = float(v)
    return float.hex(d) if d != 0 else "0.0"


def render() -> str:
    E, W, r = solve()
    w = [W[family(e)] for e in E]
    lines = []
    a = lines.append
    a("// Generated by gen_constants.py; do not edit.")
    a("// D2Q37 velocity set, quadrature weights and Hermite tables (exact doubles).")
    a("#pragma once")
    a("")
    a("namespace d2q37 {")
    a("")
    a("constexpr int Q = 37;")
    a("// integer hops e_l = (EX[l], EY[l]); lattice velocity c_l = R * e_l")
    a("constexpr int EX[Q] = {%s};" % ", ".join(str(e[0]) for e in E))
    a("constexpr int EY[Q] = {%s};" % ", ".join(str(e[1]) for e in E))
    a("// quadrature weights w_l")
    a("constexpr double W[Q] = {")
    for i in range(0, 37, 3):
        a("    " + ", ".join(hexf(v) for v in w[i:i + 3]) + ",")
    a("};")
    a("constexpr double R = %s;  // %s" % (hexf(r), mp.nstr(r, 25)))
    a("// HE[k][n] = He_n(R k), k = 0..3 (He_n(-x) = (-1)^n He_n(x))")
    a("constexpr double HE[4][5] = {")
    for k in range(4):
        a("    {" + ", ".join(hexf(hermite(n, r * k)) for n in range(5)) + "},")
    a("};")
    a("// HEF[k][n] = He_n(R k) / n!")
    a("constexpr double HEF[4][5] = {")
    for k in range(4):
        a("    {" + ", ".join(hexf(hermite(n, r * k) / mp.factorial(n)) for n in range(5)) + "},")
    a("};")
    a("// INVFAC[n] = 1 / n!")
    a("constexpr double INVFAC[5] = {%s};" % ", ".join(hexf(1 / mp.factorial(n)) for n in range(5)))
    a("// powers of r (R2 = r^2, R6_6 = r^6 / 6, IR2_3 = 3 r^-2, ...)")
    for name, v in (("R2", r ** 2), ("R4", r ** 4), ("R6", r ** 6), ("R8", r ** 8),
                    ("R6_6", r ** 6 / 6), ("R8_6", r ** 8 / 6), ("R8_24", r ** 8 / 24),
                    ("IR2", r ** -2), ("IR2_3", 3 / r ** 2), ("IR2_6", 6 / r ** 2)):
        a("constexpr double %s = %s;" % (name, hexf(v)))
    a("// sum w e_x^2, sum w e_x^4, sum w e_x^2 e_y^2")
    for name, i, j in (("G20", 2, 0), ("G40", 4, 0), ("G22", 2, 2)):
        a("constexpr double %s = %s;" % (
            name, hexf(sum(mp.mpf(float(v)) * e[0] ** i * e[1] ** j for v, e in zip(w, E)))))
    a("")
    a("}  // namespace d2q37")
    a("")
    return "\n".join(lines)


def check() -> bool:
    return os.path.exists(HEADER) and open(HEADER).read() == render()


def write() -> str:
    text = render()
    with open(HEADER, "w") as fh:
        fh.write(text)
    return HEADER


if __name__ == "__main__":
    if len(sys.argv) > 1 and sys.argv[1] == "--check":
        ok = check()
        print("up to date" if ok else "STALE")
        sys.exit(0 if ok else 1)
    print(write())
