"""Nodes and Lagrange coefficients of the binned form (sas_bins.hip).

A bin's pairs are summed as powers of v in [-1, 1]; a function of v is
replaced by the polynomial through its values at the six Gauss-Legendre nodes
v_j, the roots of P_6.  Row k, column j of the second table is the coefficient
of v^k in the Lagrange polynomial of node j.

The sums are of u^k rounded to fixed point.  Where few bits are left to u^4,
its many small values round to zero; rounding_mean gives the mean error for u
uniform on [-1, 1].

    python fit_bins.py        # prints the tables as C initialisers, and the mean
"""
import math
from fractions import Fraction

DEGREE = 6
BITS = 200  # binary digits carried by the root finding


def legendre(n):
    """Coefficients of P_n, lowest power first, as exact fractions."""
    p0, p1 = [Fraction(1)], [Fraction(0), Fraction(1)]
    for k in range(2, n + 1):
        p2 = [Fraction(0)] + [Fraction(2 * k - 1, k) * c for c in p1]
        for i, c in enumerate(p0):
            p2[i] -= Fraction(k - 1, k) * c
        p0, p1 = p1, p2
    return p1


def value(p, x):
    v = Fraction(0)
    for c in reversed(p):
        v = v * x + c
    return v


def nodes(n=DEGREE):
    """The roots of P_n in (-1, 1), ascending, by bisection of sign changes."""
    p, step = legendre(n), Fraction(1, 512)
    roots, x = [], Fraction(-1)
    while x < 1:
        a, b = x, x + step
        if value(p, a) * value(p, b) < 0:
            while b - a > Fraction(1, 1 << BITS):
                m = (a + b) / 2
                if value(p, a) * value(p, m) <= 0:
                    b = m
                else:
                    a = m
            roots.append((a + b) / 2)
        x += step
    return roots


def lagrange(v):
    """table[k][j]: coefficient of v^k in node j's Lagrange polynomial."""
    n = len(v)
    table = [[Fraction(0)] * n for _ in range(n)]
    for j in range(n):
        poly, scale = [Fraction(1)], Fraction(1)
        for i in range(n):
            if i != j:
                poly = [(poly[k - 1] if k > 0 else 0) - v[i] * (poly[k] if k < len(poly) else 0)
                        for k in range(len(poly) + 1)]
                scale *= v[j] - v[i]
        for k in range(n):
            table[k][j] = poly[k] / scale
    return table


def rounding_mean(power, bits):
    """Mean over u in [0, 1] of round(2^bits u^power) / 2^bits - u^power: the
    integer j is taken between the u where 2^bits u^power is j - 1/2 and j + 1/2."""
    scale = 2.0 ** bits
    edge = [((j + 0.5) / scale) ** (1.0 / power) for j in range(2 ** bits)] + [1.0]
    total = math.fsum(j / scale * (edge[j] - edge[j - 1]) for j in range(1, 2 ** bits + 1))
    return total - 1.0 / (power + 1)


if __name__ == "__main__":
    v = nodes()
    print("{" + ", ".join(float(x).hex() for x in v) + "}")
    for row in lagrange(v):
        print("{" + ", ".join(float(x).hex() for x in row) + "},")
    print(rounding_mean(4, 10).hex())
