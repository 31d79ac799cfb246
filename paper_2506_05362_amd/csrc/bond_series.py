"""Coefficients of the bond-law polynomial used by the step kernels.

The bond force of Sec. 3.1 needs g(x) = 1 - (1 + x)^(-1/2) with
x = (|y|^2 - |xi|^2) / |xi|^2.  For |x| <= 0.0055 the kernels evaluate
g = x * q(x) with q a polynomial of degree 6: the interpolant of
q(x) = (1 - (1 + x)^(-1/2)) / x at the Chebyshev nodes of the interval, computed
here in 80-digit decimal arithmetic.  Its constant term is exactly 1/2; with the
other coefficients rounded to double the relative error is 1.1e-18.  Up to |x| = 0.08
the kernels take a Newton step from its value.

    python paper_2506_05362_amd/csrc/bond_series.py
prints the coefficients (highest degree first, as C hex literals) and the
error of the rounded polynomial on a 801-point grid, then the largest relative
error of the Newton step, without rounding, on 0.0055 <= |x| <= 0.08.
"""
from decimal import Decimal as D, getcontext

getcontext().prec = 80
PI = D("3.14159265358979323846264338327950288419716939937510582097494459230781640628620899")


def q(x):
    if abs(x) < D(10) ** -20:
        return D("0.5") - D(3) * x / 8
    return (1 - 1 / (1 + x).sqrt()) / x


def cos(t):
    s, term, k = D(0), D(1), 0
    while abs(term) > D(10) ** -75:
        s += term
        term = -term * t * t / ((2 * k + 1) * (2 * k + 2))
        k += 1
    return s


def solve(A, b):
    n = len(b)
    for c in range(n):
        p = max(range(c, n), key=lambda i: abs(A[i][c]))
        A[c], A[p], b[c], b[p] = A[p], A[c], b[p], b[c]
        for i in range(c + 1, n):
            f = A[i][c] / A[c][c]
            for j in range(c, n):
                A[i][j] -= f * A[c][j]
            b[i] -= f * b[c]
    x = [D(0)] * n
    for i in reversed(range(n)):
        x[i] = (b[i] - sum(A[i][j] * x[j] for j in range(i + 1, n))) / A[i][i]
    return x


def coefficients(R, N):
    xs = [R * cos((2 * k + 1) * PI / (2 * N)) for k in range(N)]
    return solve([[x ** j for j in range(N)] for x in xs], [q(x) for x in xs])


def max_rel_error(cs, R):
    worst = D(0)
    for k in range(-400, 401):
        x = R * k / 400
        p = D(0)
        for c in reversed(cs):
            p = p * x + c
        worst = max(worst, abs(p - q(x)) / q(x))
    return worst


def newton_error(cs, x):
    p = D(0)
    for c in reversed(cs):
        p = p * x + c
    r = 1 - x * p
    r += r * (1 - (1 + x) * r * r) / 2
    return abs((1 - r) - x * q(x)) / abs(x * q(x))


if __name__ == "__main__":
    R, N, wide = D("0.0055"), 7, D("0.08")
    co = coefficients(R, N)
    rounded = [D(float(c)) for c in co]
    print("|x| <= %s: constant term" % R, float(co[0]))
    print("c%d..c1:" % (N - 1), ", ".join(float(c).hex() for c in reversed(co[1:])))
    print("max relative error, rounded coefficients: %.3e" % max_rel_error(rounded, R))
    grid = [s * (R + (wide - R) * k / 400) for k in range(401) for s in (1, -1)]
    print("|x| <= %s, after the Newton step: %.3e" % (wide, max(newton_error(rounded, x) for x in grid)))
