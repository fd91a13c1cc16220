"""Generate hct_cut.inc: polynomials for the part of a ball beyond a sphere.

With a descreening cutoff c the ball of radius S at distance r loses the part
outside the sphere of radius c around the atom, H(r; c, S) = J / (4 r) with
e = (r + S - c) / c and s = S / c (0 <= e <= 2 s where the ball straddles the
sphere):

    J = e - ln(1 + e) + (S - r) e^2 / (2 (r + S)) = e^2 (s A(e) - e L(e)),
    A(e) = 1 / (1 + e),   L(e) = (ln(1 + e) - e + e^2/2) / e^3
                               = 1/3 - e/4 + e^2/5 - ...

(the first form cancels to an s-th part of its terms, the second does not).
The fits are relative-weighted least squares at Chebyshev nodes in mpmath on
0 <= e <= EMAX.
"""
import os

import mpmath
import numpy as np

from gen_hct_poly import fit

EMAX = 0.36


def L_exact(e):
    e = mpmath.mpf(e)
    if e == 0:
        return mpmath.mpf(1) / 3
    return (mpmath.log(1 + e) - e + e * e / 2) / e ** 3


def A_exact(e):
    return 1 / (1 + mpmath.mpf(e))


FUNCS = {"L": L_exact, "A": A_exact}
FITS = {
    # name: (degree, C type, fma, literal suffix, digits, function)
    "hct_cut_l": (6, "float", "fmaf", "f", 9, "L"),
    "hct_cut_a": (6, "float", "fmaf", "f", 9, "A"),
    "hct_cut_l64": (14, "double", "fma", "", 17, "L"),
}


def horner_error(c, ctype, f_exact):
    dt = np.float32 if ctype == "float" else np.float64
    cd = [dt(float(v)) for v in c]
    worst = 0.0
    for e in np.linspace(0.0, EMAX, 2001):
        e = dt(e)
        p = cd[-1]
        for v in cd[-2::-1]:
            p = dt(p * e + v)
        worst = max(worst, abs(float(p) / float(f_exact(float(e))) - 1.0))
    return worst


def main():
    mpmath.mp.dps = 50
    lines = ["// Generated by gen_hct_cut.py -- do not edit.",
             "// L(e) = (ln(1 + e) - e + e^2/2) / e^3 and A(e) = 1 / (1 + e) on e in [0, %.2f]." % EMAX,
             "#define GBMC_CUT_EMAX %.2ff" % EMAX]
    for name, (deg, ctype, fma, suf, dig, fn) in FITS.items():
        c = fit(EMAX, deg, FUNCS[fn])
        err = horner_error(c, ctype, FUNCS[fn])
        lines += ["", "// %s: %s, degree %d; max relative error %.2e in %s." % (name, fn, deg, err, ctype),
                  "__device__ __forceinline__ %s %s(%s e) {" % (ctype, name, ctype),
                  "    %s p = %.*e%s;" % (ctype, dig, float(c[-1]), suf)]
        lines += ["    p = %s(p, e, %.*e%s);" % (fma, dig, float(v), suf) for v in c[-2::-1]]
        lines += ["    return p;", "}"]
        print(name, "max rel err", err)
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "hct_cut.inc"), "w") as f:
        f.write("\n".join(lines) + "\n")


if __name__ == "__main__":
    main()
