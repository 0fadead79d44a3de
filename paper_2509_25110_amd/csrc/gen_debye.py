"""Write debye_coef.hpp: the coefficients of Debye's polynomials u_k(t) (DLMF 10.41.10),
generated exactly (rational arithmetic) from their recurrence (DLMF 10.41.11)

    u_0(t) = 1,
    u_{k+1}(t) = t^2 (1 - t^2) u_k'(t) / 2 + (1/8) int_0^t (1 - 5 s^2) u_k(s) ds,

and stored as u_k(t) = t^k sum_{i=0..k} c[k][i] (t^2)^i; also a polynomial for
f(y) = sum_m y^m / (2m + 3) = (atanh(sqrt y) - sqrt y) / y^(3/2) on 0 <= y <= ETA_YMAX,
the interpolant of f in ETA_DEG + 1 Chebyshev nodes (50 digits), rounded to double.
Run from this directory: ``python gen_debye.py`` (rewrites debye_coef.hpp).
"""
import os
from fractions import Fraction

import mpmath as mp

K = 10  # terms kept after u_0
ETA_DEG = 21  # f has its singularity at y = 1: the interpolation error is below 2e-17 of f
ETA_YMAX = "0.45"


def eta_poly():
    with mp.workdps(50):
        b = mp.mpf(ETA_YMAX)
        f = lambda y: mp.nsum(lambda m: y ** int(m) / (2 * int(m) + 3), [0, 400], method="d")  # noqa: E731
        n = ETA_DEG + 1
        ys = [b * (1 + mp.cos(mp.pi * (2 * i + 1) / (2 * n))) / 2 for i in range(n)]
        A = mp.matrix(n, n)
        for i, y in enumerate(ys):
            for j in range(n):
                A[i, j] = y ** j
        c = mp.lu_solve(A, mp.matrix([f(y) for y in ys]))
        worst = max(abs(mp.polyval([c[j] for j in range(n - 1, -1, -1)], b * k / 200) / f(b * k / 200) - 1)
                    for k in range(201))
        assert worst < 2e-17, worst
        return [float(c[j]) for j in range(n)]


def polys(kmax):
    us = [[Fraction(1)]]  # coefficient lists in powers of t
    for _ in range(kmax):
        u = us[-1]
        new = [Fraction(0)] * (len(u) + 3)
        for i in range(1, len(u)):          # t^2 (1 - t^2)/2 * d/dt (c t^i) = i c (t^(i+1) - t^(i+3))/2
            c = u[i] * i
            new[i + 1] += c / 2
            new[i + 3] -= c / 2
        for i, c in enumerate(u):           # (1/8) int_0^t (1 - 5 s^2) c s^i ds
            new[i + 1] += c / (8 * (i + 1))
            new[i + 3] -= 5 * c / (8 * (i + 3))
        while new and new[-1] == 0:
            new.pop()
        us.append(new)
    return us


def main():
    us = polys(K)
    lines = ["// Generated by gen_debye.py: Debye's polynomials u_k(t), k = 1..%d (DLMF 10.41.10-11)," % K,
             "// u_k(t) = t^k * sum_{i=0..k} kDebyeC[kDebyeOff[k] + i] * t^(2 i).",
             "#pragma once", "",
             "// constant memory on the device, plain constants on the host",
             "#if defined(__HIP_DEVICE_COMPILE__)",
             "#define LOS_DEBYE_TABLE static __constant__ const",
             "#else",
             "#define LOS_DEBYE_TABLE static const",
             "#endif", "", "namespace los {", "",
             "constexpr int kDebyeK = %d;" % K,
             "constexpr int kDebyeOff[%d] = {%s};" % (K + 1, ", ".join(
                 str(sum(j + 1 for j in range(1, k))) if k > 0 else "0" for k in range(K + 1))),
             "LOS_DEBYE_TABLE double kDebyeC[] = {"]
    for k in range(1, K + 1):
        u = us[k]
        coef = [u[k + 2 * i] for i in range(k + 1)]
        assert all(u[j] == 0 for j in range(len(u)) if (j - k) % 2 or j < k)
        lines.append("    // u_%d: %s" % (k, " ".join("%s" % c for c in coef)))
        lines.append("    " + ", ".join("%.17g" % float(c) for c in coef) + ",")
    eta = eta_poly()
    lines += ["};", "",
              "// f(y) = sum_m y^m / (2 m + 3) on 0 <= y <= kEtaYMax, degree %d (relative error below 2e-17):" % ETA_DEG,
              "// atanh(s) - s = s^3 f(s^2).",
              "constexpr double kEtaYMax = %s;" % ETA_YMAX,
              "constexpr int kEtaDeg = %d;" % ETA_DEG,
              "LOS_DEBYE_TABLE double kEtaC[] = {"]
    for m0 in range(0, len(eta), 4):
        lines.append("    " + ", ".join("%.17g" % v for v in eta[m0:m0 + 4]) + ",")
    lines += ["};", "", "}  // namespace los", ""]
    out = os.path.join(os.path.dirname(os.path.abspath(__file__)), "debye_coef.hpp")
    with open(out, "w") as f:
        f.write("\n".join(lines))
    print("wrote", out)


if __name__ == "__main__":
    main()
