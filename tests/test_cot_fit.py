"""The polynomial fits of the cotangent-form step (csrc/cot_fit.hpp): for every variant,
|1 + x R(x) - sqrt(x) cot(sqrt x)| is within the header's bound on [0, X_v] (2^-57 up to degree 8,
2^-54 beyond) with the coefficients as written, checked in 40-digit arithmetic on a grid finer than
the generator's (K(0) = 1 exactly by construction)."""
import os
import re

import mpmath as mp

HDR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1704_08919_amd", "csrc",
                   "cot_fit.hpp")


def test_fits_meet_their_bound():
    mp.mp.dps = 40
    src = open(HDR).read()
    deg = [int(v) for v in re.search(r"kCotDegree\[kNumCot\] = \{([^}]*)\}", src).group(1).split(",")]
    xmax = [float(v) for v in re.search(r"kCotXmax\[kNumCot\] = \{([^}]*)\}", src).group(1).split(",")]
    body = re.search(r"kCotCoef\[kNumCot\]\[kCotMaxTerms\] = \{(.*?)\n\};", src, re.S).group(1)
    coef = [[mp.mpf(float(v)) for v in row.split(",")] for row in re.findall(r"\{([^{}]*)\}", body)]
    assert len(deg) == len(xmax) == len(coef)
    assert all(a < b for a, b in zip(xmax, xmax[1:])) and xmax[-1] < float(mp.pi ** 2)
    for n, X, c in zip(deg, xmax, coef):
        tol = mp.mpf(2) ** (-57 if n <= 8 else -54)
        assert all(v == 0 for v in c[n:])
        for i in range(1, 6001):
            x = mp.mpf(X) * i / 6000
            r = mp.mpf(0)
            for cj in reversed(c[:n]):
                r = r * x + cj
            s = mp.sqrt(x)
            assert abs(1 + x * r - s * mp.cot(s)) <= tol, (n, X, i)
