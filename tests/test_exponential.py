"""The kernels' fp64 exponential: its polynomial, worked out again in exact rational numbers, and its error."""
import os
import re
from decimal import Decimal, localcontext
from fractions import Fraction
from math import factorial

import paper_2512_23858_amd as ygg

SERIES, DEGREE = 18, 12


def _coefficients():
    """Lowest power first, as the header has them."""
    path = os.path.join(os.path.dirname(ygg.__file__), "csrc", "ygg_device.h")
    body = re.search(r"void exp_clamped_n\(.*?constexpr double c\[\] = \{(.*?)\};", open(path).read(), re.S).group(1)
    return [float(x) for x in body.split(",")][::-1]


def _half_ln2():
    with localcontext() as ctx:
        ctx.prec = 60
        return Fraction(Decimal(2).ln() / 2)


def _chebyshev(n):
    a, b = [Fraction(1)], [Fraction(0), Fraction(1)]
    for _ in range(n - 1):
        c = [Fraction(0)] + [2 * x for x in b]
        for i, x in enumerate(a):
            c[i] -= x
        a, b = b, c
    return b


def test_polynomial_is_the_economised_taylor_series():
    h = _half_ln2()
    p = [Fraction(1, factorial(i)) for i in range(SERIES + 1)]
    for n in range(SERIES, DEGREE, -1):       # x^n -> x^n - h^n T_n(x / h) / 2^(n-1): off by h^n / 2^(n-1) at most on |x| <= h
        t = _chebyshev(n)
        for i in range(n):
            p[i] -= p[n] / t[n] * t[i] * h ** (n - i)
        p.pop()
    assert _coefficients() == [float(x) for x in p]


def test_polynomial_is_no_further_off_than_the_series_of_degree_13():
    h, c = _half_ln2(), [Fraction(x) for x in _coefficients()]
    taylor = [Fraction(1.0 / factorial(i)) for i in range(14)]
    with localcontext() as ctx:
        ctx.prec = 50

        def worst(p):
            w = Decimal(0)
            for i in range(401):
                x = Fraction(round(h * (2 * Fraction(i, 400) - 1) * 2 ** 60), 2 ** 60)
                v = sum(a * x ** k for k, a in enumerate(p))
                exact = (Decimal(x.numerator) / Decimal(x.denominator)).exp()
                w = max(w, abs(Decimal(v.numerator) / Decimal(v.denominator) / exact - 1))
            return w
        assert worst(c) <= Decimal("5e-19") < worst(taylor) < Decimal("6e-18")
