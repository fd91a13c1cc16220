"""Generate hct_vfar.inc: the polynomials P and W of gen_hct_poly.py for tiles
far enough apart that every pair has y = (S/r)^2 <= YVFAR, where shorter fits are
as accurate as the ones on [0, 0.10]."""
import os

from gen_hct_poly import FUNCS, fit, horner_error

YVFAR = 0.015
FITS = {
    # name: (degree, C type, fma, literal suffix, digits, function)
    "hct_poly_vfar": (3, "float", "fmaf", "f", 9, "P"),
    "hct_w_vfar": (3, "float", "fmaf", "f", 9, "W"),
    "hct_poly64_vfar": (6, "double", "fma", "", 17, "P"),
}


def main():
    lines = ["// Generated by gen_hct_vfar.py -- do not edit.",
             "#define GBMC_HCT_YVFAR %.3ff" % YVFAR]
    for name, (deg, ctype, fma, suf, dig, fn) in FITS.items():
        c = fit(YVFAR, deg, FUNCS[fn])
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
