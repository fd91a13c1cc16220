"""The FP64 kernels' polynomial for 2^f (csrc/exp2_poly.inc) on the CPU, by
Horner's rule in double precision against 40-digit arithmetic."""
import os
import re

import mpmath
import numpy as np

INC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1803_09652_amd", "csrc", "exp2_poly.inc")


def test_fit_meets_its_stated_error():
    text = open(INC).read()
    err = float(re.search(r"max relative error ([\d.e+-]+) in double", text).group(1))
    coef = [float(v) for v in re.findall(r"([-+]?\d\.\d+e[-+]\d+)[;)]", text)]
    assert len(coef) == 12 and coef[-1] == 1.0
    mpmath.mp.dps = 40
    worst = 0.0
    for x in np.linspace(-0.5, 0.5, 1501):
        p = coef[0]
        for v in coef[1:]:
            p = p * float(x) + v
        worst = max(worst, abs(float(mpmath.mpf(p) / mpmath.power(2, mpmath.mpf(float(x))) - 1)))
    assert worst <= 1.1 * err and err < 2.3e-16


def test_fused_error_is_near_that_of_rounding():
    # with fused operations, as the kernels evaluate it, no further off than 1.06 units
    # of 2^-53 (2^f itself, rounded: 1.00)
    from fractions import Fraction
    coef = [float(v) for v in re.findall(r"([-+]?\d\.\d+e[-+]\d+)[;)]", open(INC).read())]
    mpmath.mp.dps = 40
    worst = 0.0
    for x in np.random.default_rng(1).uniform(-0.5, 0.5, 3000):
        p = coef[0]
        for v in coef[1:]:
            p = float(Fraction(p) * Fraction(float(x)) + Fraction(v))   # one rounding
        worst = max(worst, abs(float(mpmath.mpf(p) / mpmath.power(2, mpmath.mpf(float(x))) - 1)))
    assert worst <= 1.06 * 2.0 ** -53
