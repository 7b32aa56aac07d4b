"""Fits the polynomial approximations used by the SIE deflection kernels.

atan(u) = u * A(u^2) on |u| <= 1/sqrt(3) and on |u| <= 1, and atanh(v) = v * B(v^2)
on |v| <= 1/2, with A and B the polynomials of least maximum relative error
found by the Remez exchange algorithm (Remez 1934) in double precision, with
the constant coefficient held at exactly 1. A free constant coefficient would
come out 1 - O(1e-8) and round to 1.0 in float32, which shifts the whole
equioscillating error curve to one side: a bias of the same sign at every
subsample, which sums coherently over an image. With it pinned the error
oscillates about zero. Run it to regenerate the coefficient table in sie_poly.h:

    python fit_minimax.py > sie_poly.h
"""
import numpy as np


def remez_relative_c0(f, a, b, degree, iters=80):
    """p(s) = 1 + c_1 s + ... + c_degree s^degree minimising max |p/f - 1| on [a, b]."""
    m = degree + 1                     # unknowns c_1..c_degree and the level E
    k = np.arange(m)
    x = 0.5 * (a + b) + 0.5 * (a - b) * np.cos(np.pi * k / (m - 1))
    x[0] = a + (b - a) * 1e-3          # the error vanishes at s = 0 itself
    grid = np.linspace(a + (b - a) * 1e-6, b, 400001)
    fg = f(grid)
    c = None
    for _ in range(iters):
        fx = f(x)
        A = np.zeros((m, m))
        for j in range(1, degree + 1):
            A[:, j - 1] = x ** j
        A[:, -1] = -((-1.0) ** k) * fx     # p(x_k) - f(x_k) = (-1)^k E f(x_k)
        sol = np.linalg.solve(A, fx - 1.0)
        c = np.concatenate([[1.0], sol[:-1]])
        err = np.polyval(c[::-1], grid) / fg - 1.0
        # new reference: one extremum of the error in each sign-alternating segment
        sign = np.sign(err)
        idx = np.nonzero(np.diff(sign) != 0)[0]
        bounds = np.concatenate([[0], idx + 1, [len(grid)]])
        ext = np.array([lo + int(np.argmax(np.abs(err[lo:hi]))) for lo, hi in zip(bounds[:-1], bounds[1:]) if hi > lo])
        if len(ext) < m:
            break
        while len(ext) > m:              # drop the smaller end extremum
            ext = ext[1:] if abs(err[ext[0]]) < abs(err[ext[-1]]) else ext[:-1]
        x = grid[ext]
    c32 = np.asarray(c, np.float32).astype(np.float64)
    e32 = np.polyval(c32[::-1], grid) / fg - 1.0
    return c, float(np.max(np.abs(e32))), float(np.mean(e32))


def atan_over_u(s):
    s = np.asarray(s, dtype=np.float64)
    r = np.sqrt(np.maximum(s, 1e-300))
    return np.where(s > 0, np.arctan(r) / r, 1.0)


def atanh_over_v(s):
    s = np.asarray(s, dtype=np.float64)
    r = np.sqrt(np.maximum(s, 1e-300))
    return np.where(s > 0, np.arctanh(r) / r, 1.0)


def emit(name, coeffs, err, mean, domain):
    print(f"// {name}: max relative error {err:.3e} (mean {mean:+.1e}) on {domain}, float32 coefficients")
    print(f"#define {name}_DEGREE {len(coeffs) - 1}")
    body = ", ".join(f"{float(v)!r}" for v in coeffs)
    print(f"static constexpr double {name}_D[{len(coeffs)}] = {{{body}}};")


if __name__ == "__main__":
    print("// Generated by fit_minimax.py -- coefficients in increasing powers of s.")
    print("#pragma once")
    cs, es, ms = remez_relative_c0(atan_over_u, 0.0, 1.0001 / 3.0, 5)
    emit("ATAN_SMALL_POLY", cs, es, ms, "s = u^2 in [0, 1/3]")
    ca, ea, ma = remez_relative_c0(atan_over_u, 0.0, 1.0001, 8)
    emit("ATAN_UNIT_POLY", ca, ea, ma, "s = u^2 in [0, 1]")
    cb, eb, mb = remez_relative_c0(atanh_over_v, 0.0, 0.2501, 5)
    emit("ATANH_POLY", cb, eb, mb, "s = v^2 in [0, 1/4]")
