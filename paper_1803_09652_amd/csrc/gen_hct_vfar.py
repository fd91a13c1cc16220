"""Generate hct_vfar.inc: the polynomials P and W of gen_hct_poly.py for tiles
far enough apart that every pair has y = (S/r)^2 <= YVFAR, where shorter fits are
as accurate as the ones on [0, 0.10].

The FP64 fit is rounded one coefficient after the other, from the constant up, the
rest fitted anew to what the rounded ones leave.  Rounded all at once its constant
came out a unit above 1/3: with fused operations, largest and mean errors of 1.74
and 0.73 units of 2^-53 on [0, 0.015], now 1.28 and 0.42, against 1.46 and 0.61
of the degree-10 fit on [0, 0.10]."""
import os

import mpmath

from gen_hct_poly import FUNCS, fit, horner_error

YVFAR = 0.015
FITS = {
    # name: (degree, C type, fma, literal suffix, digits, function)
    "hct_poly_vfar": (3, "float", "fmaf", "f", 9, "P"),
    "hct_w_vfar": (3, "float", "fmaf", "f", 9, "W"),
    "hct_poly64_vfar": (6, "double", "fma", "", 17, "P"),
}


def fit_rounded(ymax, deg, f_exact):
    """fit(), with coefficients rounded to double one by one from the constant up."""
    mpmath.mp.dps = 50
    m = 200
    ys = [(mpmath.cos(mpmath.pi * (k + mpmath.mpf(1) / 2) / m) + 1) / 2 * mpmath.mpf(ymax) for k in range(m)]
    fs = [f_exact(y) for y in ys]
    done = []
    while len(done) <= deg:
        A, b = mpmath.matrix(m, deg + 1 - len(done)), mpmath.matrix(m, 1)
        for i, (y, f) in enumerate(zip(ys, fs)):
            for j in range(len(done), deg + 1):
                A[i, j - len(done)] = y ** j / f
            b[i] = 1 - mpmath.fsum(mpmath.mpf(c) * y ** j for j, c in enumerate(done)) / f
        # the first is the value at 0 (1/3); the fit alone would miss it by an ulp
        done.append(float(f_exact(0) if not done else mpmath.lu_solve(A.T * A, A.T * b)[0]))
    return done


def main():
    lines = ["// Generated by gen_hct_vfar.py -- do not edit.",
             "#define GBMC_HCT_YVFAR %.3ff" % YVFAR]
    for name, (deg, ctype, fma, suf, dig, fn) in FITS.items():
        c = (fit_rounded if ctype == "double" else fit)(YVFAR, deg, FUNCS[fn])
        err = horner_error(c, YVFAR, ctype, FUNCS[fn])
        lines += ["", "// %s: %s, degree %d on y in [0, %.3f]; max relative error %.2e in %s." % (
                      name, fn, deg, YVFAR, err, ctype),
                  "__device__ __forceinline__ %s %s(%s y) {" % (ctype, name, ctype),
                  "    %s p = %.*e%s;" % (ctype, dig, float(c[-1]), suf)]
        lines += ["    p = %s(p, y, %.*e%s);" % (fma, dig, float(v), suf) for v in c[-2::-1]]
        lines += ["    return p;", "}"]
        print(name, "max rel err", err)
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "hct_vfar.inc"), "w") as f:
        f.write("\n".join(lines) + "\n")


if __name__ == "__main__":
    main()
