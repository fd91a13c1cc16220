"""The fits of tiles far apart (csrc/hct_vfar.inc) on the CPU: each polynomial
by Horner's rule in its own precision against the Taylor series of
P(y) = sum_{k>=1} k y^(k-1) / (2k + 1) and the closed form W(y) = (1 - y)^-2 in
40-digit arithmetic, over its domain and no worse than the fits of the nearer
tiles that they take the place of (csrc/hct_poly.inc)."""
import os
import re

import mpmath
import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1803_09652_amd", "csrc")
PATTERN = re.compile(r"// (\w+): ([PW]), degree (\d+) on y in \[0, ([\d.]+)\]; max relative "
                     r"error ([\d.e+-]+) in (float|double)\.\n(?:#define \w+ [\d.]+f?\n)?"
                     r"__device__ __forceinline__ \w+ \1\(\w+ y\) \{\n(.*?)\n    return p;", re.S)


def fits(name):
    text = open(os.path.join(CSRC, name)).read()
    return text, {m.group(1): (m.group(2), float(m.group(4)), float(m.group(5)), m.group(6),
                               [float(v) for v in re.findall(r"([-+]?\d\.\d+e[-+]\d+)f?", m.group(7))])
                  for m in PATTERN.finditer(text)}


TEXT, VFAR = fits("hct_vfar.inc")
FAR = fits("hct_poly.inc")[1]


def exact(fn, y):
    mpmath.mp.dps = 40
    y = mpmath.mpf(y)
    if fn == "W":
        return 1 / (1 - y) ** 2
    return mpmath.fsum(k * y ** (k - 1) / (2 * k + 1) for k in range(1, 40))


@pytest.mark.parametrize("name,far", [("hct_poly_vfar", "hct_poly_far"), ("hct_w_vfar", "hct_w_far"),
                                      ("hct_poly64_vfar", "hct_poly64_far")])
def test_fit_meets_its_stated_error(name, far):
    fn, ymax, err, ctype, coef = VFAR[name]
    assert ymax == float(re.search(r"#define GBMC_HCT_YVFAR ([\d.]+)f", TEXT).group(1))
    dt = np.float32 if ctype == "float" else np.float64
    worst = 0.0
    for y in np.linspace(0.0, ymax, 1201):
        p = dt(coef[0])
        for v in coef[1:]:
            p = dt(dt(p * dt(y)) + dt(v))
        worst = max(worst, abs(float(p) / float(exact(fn, float(dt(y)))) - 1.0))
    assert worst <= 1.01 * err + 1e-18
    # half a unit in the last place of a value just above a power of two, and
    # another of the last product and sum
    assert err <= max(FAR[far][2], 2.0 ** -23 if ctype == "float" else 2.0 ** -52)


def test_fp64_fit_is_no_less_accurate_than_the_one_it_replaces():
    # with fused operations, as the kernels evaluate both: largest and mean errors on the
    # domain, in exact arithmetic
    from fractions import Fraction

    def errors(coef, ys):
        out = []
        for y in ys:
            p = coef[0]
            for v in coef[1:]:
                p = float(Fraction(p) * Fraction(y) + Fraction(v))      # one rounding
            out.append(abs(float(mpmath.mpf(p) / exact("P", y) - 1)))
        return max(out), sum(out) / len(out)
    ys = [float(v) for v in np.random.default_rng(0).uniform(0.0, VFAR["hct_poly64_vfar"][1], 1500)]
    new, old = (errors(f[4], ys) for f in (VFAR["hct_poly64_vfar"], FAR["hct_poly64_far"]))
    assert new[0] <= old[0] and new[1] <= old[1], (new, old)
