"""Coefficients of the float64 atan and atanh of the general models (model.hip).

With F(z) = sum_k z^k / (2k + 1), atan(w) = w F(-w^2) and atanh(w) = w F(w^2). F is
written 1 + z G(z), the leading 1 exact, and G as its Chebyshev interpolant, in
60-digit arithmetic, turned into powers of z: on [-tan(pi/8)^2, 0] for the atan
(arguments reduced to |w| <= tan(pi/8)), and on [-0.053, 1/9] for the atanh
(|w| <= 1/3) and the series of nearly round lenses. Prints the tables with the
largest error of F over 400 points, the coefficients rounded to float64:

    python fit_atan64.py
"""
from decimal import Decimal as D
from decimal import getcontext

getcontext().prec = 60
PI = D("3.14159265358979323846264338327950288419716939937510582097494459")
EPS = D(10) ** -58


def cos(x):
    x = x % (2 * PI)
    t = s = D(1)
    k = 0
    while abs(t) > EPS:
        k += 2
        t = -t * x * x / (k * (k - 1))
        s += t
    return s


def F(z):
    s, p, k = D(0), D(1), 0
    while abs(p) > EPS or k < 3:
        s += p / (2 * k + 1)
        p *= z
        k += 1
    return s


def G(z):
    return (F(z) - 1) / z if abs(z) > D(10) ** -25 else D(1) / 3


def interpolant(f, a, b, degree):
    """Powers of z of the Chebyshev series of f on [a, b], cut at `degree`."""
    n = degree + 12
    mid, half = (a + b) / 2, (b - a) / 2
    nodes = [cos(PI * (2 * i + 1) / (2 * n)) for i in range(n)]
    values = [f(mid + half * x) for x in nodes]
    c = [sum(v * cos(PI * j * (2 * i + 1) / (2 * n)) for i, v in enumerate(values)) * 2 / n for j in range(degree + 1)]
    c[0] /= 2
    powers = [D(0)] * (degree + 1)      # in t = (z - mid) / half
    t0, t1 = [D(1)], [D(0), D(1)]
    for j in range(degree + 1):
        for i, v in enumerate(t0):
            powers[i] += c[j] * v
        t2 = [D(0)] + [2 * v for v in t1]
        for i, v in enumerate(t0):
            t2[i] -= v
        t0, t1 = t1, t2
    out, q = [D(0)] * (degree + 1), [D(1)]
    for v in powers:
        for k, u in enumerate(q):
            out[k] += v * u
        nxt = [D(0)] * (len(q) + 1)
        for k, u in enumerate(q):
            nxt[k + 1] += u / half
            nxt[k] -= u * mid / half
        q = nxt
    return [float(v) for v in out]


if __name__ == "__main__":
    for name, a, b in (("ATAN64", "-0.17157287525381", "0"), ("ATANH64", "-0.0530", "0.1112")):
        a, b = D(a), D(b)
        co = interpolant(G, a, b, 10)
        worst = D(0)
        for i in range(400):
            z = a + (b - a) * i / 399
            s = D(0)
            for v in reversed(co):
                s = s * z + D(v)
            worst = max(worst, abs(z * s + 1 - F(z)))
        print(f"// {name}: G on [{a}, {b}], largest error of F {float(worst):.1e}")
        print(f"static constexpr double {name}[11] = {{{', '.join(repr(v) for v in co)}}};")
