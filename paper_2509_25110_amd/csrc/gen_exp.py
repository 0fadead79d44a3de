"""The polynomial of the emulator's exp (kExpQ in emu_gemm.hip): q(r) = (e^r - 1 - r) / r^2 on
|r| <= ln 2 / 2, as the interpolant of degree DEG in Chebyshev nodes (50 digits), rounded to
double.  ``python gen_exp.py`` prints the coefficients, constant term first."""
import mpmath as mp

DEG = 10  # error 3.4e-19 of e^r (Taylor's polynomial needs a term more for 5.7e-18)


def coefficients():
    with mp.workdps(50):
        b = mp.log(2) / 2 * (1 + mp.mpf(2) ** -20)
        f = lambda r: mp.nsum(lambda m: r ** int(m) / mp.factorial(int(m) + 2), [0, 40], method="d")  # noqa: E731
        n = DEG + 1
        xs = [b * mp.cos(mp.pi * (2 * i + 1) / (2 * n)) for i in range(n)]
        A = mp.matrix(n, n)
        for i, x in enumerate(xs):
            for j in range(n):
                A[i, j] = x ** j
        c = [float(v) for v in mp.lu_solve(A, mp.matrix([f(x) for x in xs]))]
        worst = max(abs(r * r * (mp.polyval(c[::-1], r) - f(r))) / mp.exp(r)
                    for r in (b * k / 500 for k in range(-500, 501)))
        return c, worst


if __name__ == "__main__":
    c, worst = coefficients()
    print("largest error, relative to e^r: %s" % mp.nstr(worst, 3))
    print(", ".join("%.17g" % v for v in c))
