"""Polynomials of the Sersic constant b_n (prologue.hip).

b_n is the root of P(2n, b) = 1/2 (R_e is the half-light radius). Its only
singularity near the accepted range 0.2 <= n <= 10 is n = 0, so on quarters of an
octave of n, [2^e (1 + s/4), 2^e (1 + (s + 1)/4)], the Chebyshev series falls by about
18 per degree in the first quarter and faster in the others. Each piece's series is
cut at DEGREE, in 50-digit arithmetic, and turned into powers of t in [-1, 1]. Writes
bn_poly.h and prints the largest relative errors of b_n and of db_n/dn as evaluated in
float64:

    python fit_bn.py
"""
import os
import random
from decimal import Decimal as D
from decimal import getcontext

from fit_atan64 import PI, cos

getcontext().prec = 50
E_MIN, E_MAX, DEGREE = -3, 3, 13    # pieces from 0.125 up to 16
LN2PI = (2 * PI).ln()


def lgamma(z):
    """ln Gamma(z): the recurrence up to z >= 40, then Stirling's series (A&S 6.1.41)."""
    shift = D(0)
    while z < 40:
        shift += z.ln()
        z += 1
    b = [D(1) / 6, D(-1) / 30, D(1) / 42, D(-1) / 30, D(5) / 66, D(-691) / 2730, D(7) / 6, D(-3617) / 510,
         D(43867) / 798, D(-174611) / 330, D(854513) / 138, D(-236364091) / 2730, D(8553103) / 6]
    s = sum(v / (2 * k * (2 * k - 1) * z ** (2 * k - 1)) for k, v in enumerate(b, 1))
    return (z - D("0.5")) * z.ln() - z + LN2PI / 2 + s - shift


def bn(n):
    """Newton's iteration on the power series of P(a, b), a = 2n."""
    a = 2 * n
    lg = lgamma(a + 1)
    b = max(a - D(1) / 3 + D("0.0098765") / n, a / 8)
    for _ in range(100):
        pref = (a * b.ln() - b - lg).exp()
        term = total = D(1)
        k = 0
        while term > D(10) ** -48 * total:
            k += 1
            term *= b / (a + k)
            total += term
        step = (pref * total - D("0.5")) / (pref * a / b)
        nb = b - step
        b = nb if nb > 0 else b / 2
        if abs(step) < D(10) ** -40 * b:
            return b
    raise RuntimeError(n)


def piece(e, s):
    """Powers of t = (n - middle) / half of the piece's Chebyshev series."""
    lo, half = D(2) ** e * (1 + D(s) / 4), D(2) ** e / 8
    m = DEGREE + 8
    nodes = [cos(PI * (2 * i + 1) / (2 * m)) for i in range(m)]
    values = [bn(lo + half * (1 + x)) for x in nodes]
    c = [sum(v * cos(PI * j * (2 * i + 1) / (2 * m)) for i, v in enumerate(values)) * 2 / m for j in range(DEGREE + 1)]
    c[0] /= 2
    powers = [D(0)] * (DEGREE + 1)
    t0, t1 = [D(1)], [D(0), D(1)]
    for j in range(DEGREE + 1):
        for i, v in enumerate(t0):
            powers[i] += c[j] * v
        t2 = [D(0)] + [2 * v for v in t1]
        for i, v in enumerate(t0):
            t2[i] -= v
        t0, t1 = t1, t2
    return [float(v) for v in powers]


def evaluate(table, n):
    """b_n and db_n/dn in float64, as the kernel takes them."""
    e = E_MIN
    while n >= 2.0 ** (e + 1):
        e += 1
    s = int((n / 2.0 ** e - 1.0) * 4.0)
    t = (n - 2.0 ** e * (1.125 + 0.25 * s)) * 8.0 * 2.0 ** -e
    c = table[4 * (e - E_MIN) + s]
    v, d = c[DEGREE], 0.0
    for k in range(DEGREE - 1, -1, -1):
        d = d * t + v
        v = v * t + c[k]
    return v, d * 8.0 * 2.0 ** -e


if __name__ == "__main__":
    table = [piece(e, s) for e in range(E_MIN, E_MAX + 1) for s in range(4)]
    rows = ",\n".join("    {" + ", ".join(repr(v) for v in r) + "}" for r in table)
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "bn_poly.h"), "w") as f:
        f.write(f"""// bn_poly.h -- generated by fit_bn.py: b_n on quarters of the octaves of n from
// 2^{E_MIN} up to 2^{E_MAX + 1}, powers of t in [-1, 1] from the piece's middle.
#pragma once

namespace lensed {{
constexpr int BN_E_MIN = {E_MIN}, BN_DEGREE = {DEGREE}, BN_PIECES = {len(table)};
__device__ const double BN_POLY[BN_PIECES][BN_DEGREE + 1] = {{
{rows}}};
}}  // namespace lensed
""")
    rng = random.Random(1)
    worst_b = worst_d = 0.0
    for n in [0.2, 0.25, 0.5, 1.0, 2.0, 4.0, 8.0, 10.0] + [0.2 * 50 ** rng.random() for _ in range(300)]:
        b, d = evaluate(table, n)
        h = D(n) / 10 ** 10
        slope = (bn(D(n) + h) - bn(D(n) - h)) / (2 * h)
        exact = bn(D(n))
        worst_b = max(worst_b, float(abs(D(b) - exact) / exact))
        worst_d = max(worst_d, float(abs(D(d) - slope) / slope))
    print(f"largest relative error: b_n {worst_b:.1e}, db_n/dn {worst_d:.1e}")
