"""The FP64 polynomials of the node phasors (csrc/gw_trig_fit.h) against sin and
cos: the errors their header states, in Horner form as the kernel evaluates it."""
import os
import re

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
PATH = os.path.join(os.path.dirname(HERE), "paper_2607_28265_amd", "csrc", "gw_trig_fit.h")


def test_trig_fit_errors():
    s, c = (np.array([float.fromhex(v) for v in g.split(",")])
            for g in re.findall(r"\{(-?0x[^{}]*)\}", open(PATH).read()))
    assert len(s) == len(c) == 8
    r = np.linspace(-0.5, 0.5, 400001)
    a, b = np.zeros_like(r), np.zeros_like(r)
    for k in range(7, -1, -1):
        a = a * r * r + s[k]
        b = b * r * r + c[k]
    # rounding of the sums adds a few units of 1e-16
    assert np.max(np.abs(r * a - np.sin(2.0 * np.pi * r))) < 2.15e-11
    assert np.max(np.abs(b - np.cos(2.0 * np.pi * r))) < 1.25e-10
