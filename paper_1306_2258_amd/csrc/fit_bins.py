"""Nodes and Lagrange coefficients of the binned form (sas_bins.hip).

A bin's pairs are summed as powers of v in [-1, 1]; a function of v is
replaced by the polynomial through its values at the six Gauss-Legendre nodes
v_j, the roots of P_6.  Row k, column j of the second table is the coefficient
of v^k in the Lagrange polynomial of node j.

    python fit_bins.py        # prints both as C initialisers
"""
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


if __name__ == "__main__":
    v = nodes()
    print("{" + ", ".join(float(x).hex() for x in v) + "}")
    for row in lagrange(v):
        print("{" + ", ".join(float(x).hex() for x in row) + "},")
