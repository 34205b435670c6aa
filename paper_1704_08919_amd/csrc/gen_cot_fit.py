"""Writes cot_fit.hpp: polynomial fits of R(x) = (K(x) - 1)/x, K(x) = sqrt(x) cot(sqrt x), for the
cotangent form of the exact midpoint step (K = 1 + x R keeps K(0) = 1 exactly).

For each degree n of K (R of degree n - 1), R is interpolated at the n Chebyshev points of
[0, X_n] in 50-digit arithmetic, its coefficients are rounded to double, and X_n is the largest
end point (bisection, rounded down to four significant digits) at which
|1 + x R_double(x) - K(x)| is within the bound on a dense grid of [0, X_n].  The bound is 2^-57 up
to degree 8.  Beyond, the rounding of the coefficients themselves (2^-55 x and more) sets a larger
one, 2^-54: those ranges are the ones that otherwise need angle halvings, whose own rounding is
larger still.  The angle error of a step is |dK| / (K^2 + x) <= |dK| of the angle, K^2 + x >= 1.

Run: python gen_cot_fit.py  (needs mpmath; the output is committed)."""
import math
import os

import mpmath as mp

mp.mp.dps = 50
FITS = [(n, mp.mpf(2) ** -57) for n in range(3, 9)] + [(n, mp.mpf(2) ** -54) for n in (10, 12, 15)]
GRID = 4001


def K(x):
    x = mp.mpf(x)
    if x == 0:
        return mp.mpf(1)
    r = mp.sqrt(x)
    return r * mp.cot(r)


def R(x):
    x = mp.mpf(x)
    if x == 0:
        return -mp.mpf(1) / 3
    return (K(x) - 1) / x


def fit(n, X):
    """Coefficients (low to high) of R of degree n - 1 interpolating at n Chebyshev points of [0, X]."""
    X = mp.mpf(X)
    nodes = [X / 2 * (1 - mp.cos(mp.pi * (2 * k + 1) / (2 * n))) for k in range(n)]
    A = mp.matrix([[t ** j for j in range(n)] for t in nodes])
    c = mp.lu_solve(A, mp.matrix([R(t) for t in nodes]))
    return [float(v) for v in c]  # rounded to double


def err(coef, X, pts=GRID):
    X, e = mp.mpf(X), mp.mpf(0)
    for i in range(pts):
        t = X * i / (pts - 1)
        r = mp.mpf(0)
        for cj in reversed(coef):
            r = r * t + mp.mpf(cj)
        e = max(e, abs(1 + t * r - K(t)))
    return e


def xmax(n, tol):
    lo, hi = mp.mpf("0.00005"), mp.mpf("5")
    for _ in range(30):
        mid = (lo + hi) / 2
        if err(fit(n, mid), mid, 401) <= tol:
            lo = mid
        else:
            hi = mid
    q = 10 ** (math.floor(math.log10(float(lo))) - 3)
    digits = math.floor(float(lo) / q)
    while True:
        X = float(f"{digits * q:.4g}")
        c = fit(n, X)
        e = err(c, X)
        if e <= tol:
            return X, c, e
        digits -= 1


def main():
    rows = []
    for n, tol in FITS:
        X, c, e = xmax(n, tol)
        rows.append((n, X, c))
        print(n, X, float(e) * 2.0 ** 57, flush=True)
    out = os.path.join(os.path.dirname(os.path.abspath(__file__)), "cot_fit.hpp")
    width = max(r[0] for r in rows)
    with open(out, "w") as fh:
        fh.write("// Generated by gen_cot_fit.py: fits of R(x) = (sqrt(x) cot(sqrt x) - 1)/x on [0, X_v]; the\n")
        fh.write("// cotangent-form step uses K = 1 + x R.  Variant v: R of degree kCotDegree[v] - 1,\n")
        fh.write("// |K_fit - K| <= 2^-57 (degree <= 8) or 2^-54 on [0, kCotXmax[v]] with the coefficients as written.\n")
        fh.write("#pragma once\n\nnamespace po {\nnamespace {\n\n")
        fh.write(f"constexpr int kNumCot = {len(rows)};\n")
        fh.write("constexpr int kCotDegree[kNumCot] = {" + ", ".join(str(r[0]) for r in rows) + "};\n")
        fh.write("constexpr double kCotXmax[kNumCot] = {" + ", ".join(repr(r[1]) for r in rows) + "};\n")
        fh.write(f"constexpr int kCotMaxTerms = {width};\n")
        fh.write("// R coefficients, constant term first (unused entries 0)\n")
        fh.write("constexpr double kCotCoef[kNumCot][kCotMaxTerms] = {\n")
        for n, X, c in rows:
            fh.write("    {" + ", ".join([repr(x) for x in c] + ["0.0"] * (width - n)) + "},\n")
        fh.write("};\n\n}  // namespace\n}  // namespace po\n")
    print("wrote", out)


if __name__ == "__main__":
    main()
