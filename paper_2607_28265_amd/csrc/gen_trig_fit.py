"""Writes gw_trig_fit.h: polynomials of the medium-accuracy sine and cosine of
a phase in cycles, used by the mixed form at the interpolation nodes.

With r in [-1/2, 1/2] and s = r^2,
  sin(2 pi r) ~ r sum_k a_k s^k,   cos(2 pi r) ~ sum_k b_k s^k,
both the Chebyshev interpolants in s (mpmath, 40 digits), converted to powers
of s and rounded to FP64.  Run from the repository root:
    python paper_2607_28265_amd/csrc/gen_trig_fit.py
"""
import os

import mpmath as mp
import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
mp.mp.dps = 40
DEG_SIN, DEG_COS = 7, 7  # degrees in s


def cheb_fit(fun, deg):
    """Coefficients in powers of s of the interpolant at the Chebyshev nodes of [0, 1/4]."""
    n = deg + 1
    s = [(1 + mp.cos(mp.pi * (2 * j + 1) / (2 * n))) / 8 for j in range(n)]
    A = mp.matrix(n, n)
    for i in range(n):
        for j in range(n):
            A[i, j] = s[i] ** j
    return list(mp.lu_solve(A, mp.matrix([fun(v) for v in s])))


def sin_over_r(s):
    r = mp.sqrt(s)
    return mp.sin(2 * mp.pi * r) / r if r else 2 * mp.pi


def error(c, fun, odd):
    r = np.linspace(0.0, 0.5, 20001)
    s = r * r
    p = np.zeros_like(r)
    for a in reversed(c):
        p = p * s + float(a)
    return float(np.max(np.abs((p * r if odd else p) - fun(2.0 * np.pi * r))))


def main():
    a = cheb_fit(sin_over_r, DEG_SIN)
    b = cheb_fit(lambda s: mp.cos(2 * mp.pi * mp.sqrt(s)), DEG_COS)
    ea, eb = error(a, np.sin, True), error(b, np.cos, False)
    row = lambda c: ", ".join(float(v).hex() for v in c)  # noqa: E731
    lines = [
        "// Generated by gen_trig_fit.py; do not edit.",
        "// sin(2 pi r) = r sum_k s[k] r^2k and cos(2 pi r) = sum_k c[k] r^2k, |r| <= 1/2",
        f"// (largest absolute errors {ea:.1e} and {eb:.1e}).",
        "#pragma once",
        "namespace gw {",
        "struct TrigFit {",
        f"  double s[{len(a)}];",
        f"  double c[{len(b)}];",
        "};",
        "inline TrigFit make_trig_fit() {",
        "  return TrigFit{",
        "      {" + row(a) + "},",
        "      {" + row(b) + "}};",
        "}",
        "}  // namespace gw",
        "",
    ]
    with open(os.path.join(HERE, "gw_trig_fit.h"), "w") as f:
        f.write("\n".join(lines))
    print(ea, eb)


if __name__ == "__main__":
    main()
