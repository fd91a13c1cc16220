"""The fits of csrc/hct_cut.inc (the part of a straddling ball beyond the
descreening sphere) on the CPU: each polynomial by Horner's rule in its own
precision against 40-digit arithmetic, and J = e^2 (s A - e L) against its
defining form e - ln(1 + e) + (S - r) e^2 / (2 (r + S))."""
import os
import re

import mpmath
import numpy as np
import pytest

INC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1803_09652_amd", "csrc", "hct_cut.inc")
TEXT = open(INC).read()
EMAX = float(re.search(r"#define GBMC_CUT_EMAX ([\d.]+)f", TEXT).group(1))
FITS = {m.group(1): (m.group(2), float(m.group(3)), m.group(4),
                     [float(v) for v in re.findall(r"([-+]?\d\.\d+e[-+]\d+)f?", m.group(5))])
        for m in re.finditer(r"// (\w+): ([LA]), degree \d+; max relative error ([\d.e+-]+) in (float|double)\."
                             r"\n.*?\{\n(.*?)\n    return p;", TEXT, re.S)}


def exact(fn, e):
    mpmath.mp.dps = 40
    e = mpmath.mpf(e)
    if fn == "A":
        return 1 / (1 + e)
    return mpmath.mpf(1) / 3 if e == 0 else (mpmath.log(1 + e) - e + e * e / 2) / e ** 3


@pytest.mark.parametrize("name", ["hct_cut_l", "hct_cut_a", "hct_cut_l64"])
def test_fit_meets_its_stated_error(name):
    fn, err, ctype, coef = FITS[name]
    dt = np.float32 if ctype == "float" else np.float64
    worst = 0.0
    for e in np.linspace(0.0, EMAX, 901):
        p = dt(coef[0])
        for v in coef[1:]:
            p = dt(dt(p * dt(e)) + dt(v))
        worst = max(worst, abs(float(p) / float(exact(fn, float(dt(e)))) - 1.0))
    assert worst <= 1.01 * err + 1e-18
    assert err < (1.5e-7 if ctype == "float" else 3e-16)


def test_reduced_form_is_the_defining_one():
    mpmath.mp.dps = 40
    for r, S, c in ((14.2, 1.4, 15.0), (15.9, 1.2, 15.0), (9.0, 1.7, 9.6), (24.9, 0.9, 25.0)):
        r, S, c = mpmath.mpf(r), mpmath.mpf(S), mpmath.mpf(c)
        e = (r + S - c) / c
        J = e - mpmath.log(1 + e) + (S - r) * e ** 2 / (2 * (r + S))
        assert abs(e ** 2 * (S / c * exact("A", e) - e * exact("L", e)) / J - 1) < 1e-30
