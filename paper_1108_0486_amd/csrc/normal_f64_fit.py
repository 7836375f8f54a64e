"""Coefficients of the FP64 logarithm, sine and cosine in xg_normal_f64.h.

  ln((1 + s) / (1 - s)) = 2 s + s z Q(z), z = s^2, |s| <= (sqrt 2 - 1) / (sqrt 2 + 1);
  sin(pi f) = f (pi + t S(t)) and cos(pi f) = 1 + t C(t), t = f^2, |f| <= 1/4.

Q, S and C interpolate their functions at the Chebyshev nodes of the argument's
range, computed with 60-digit decimals from the Taylor series and rounded to
double at the end.  Prints the coefficients (constant term first) as C double
literals and the largest relative error of the whole formula on a grid, for
the unrounded coefficients.
Run: python3 normal_f64_fit.py
"""
from decimal import Decimal as D
from decimal import getcontext
from fractions import Fraction
import math

getcontext().prec = 60


def pi():
    """Machin: pi = 16 atan(1/5) - 4 atan(1/239)."""
    def atan_inv(q):
        x = D(1) / q
        total, power, k = D(0), x, 0
        while abs(power) > D(10) ** -58:
            total += power / (2 * k + 1) * (1 if k % 2 == 0 else -1)
            power /= q * q
            k += 1
        return total
    return 16 * atan_inv(5) - 4 * atan_inv(239)


PI = pi()


def series(coef, x):
    total, power, k = D(0), D(1), 0
    while k < 80:
        total += coef(k) * power
        power *= x
        k += 1
    return total


def q_exact(z):   # (atanh-series - 2) / z: 2 / 3 + 2 z / 5 + ...
    return series(lambda k: D(2) / (2 * k + 3), z)


def s_exact(t):   # (sin(pi f) / f - pi) / t
    return series(lambda k: (-1) ** (k + 1) * PI ** (2 * k + 3) / math.factorial(2 * k + 3), t)


def c_exact(t):   # (cos(pi f) - 1) / t
    return series(lambda k: (-1) ** (k + 1) * PI ** (2 * k + 2) / math.factorial(2 * k + 2), t)


def interpolate(fn, top, terms):
    """Monomial coefficients of the polynomial through fn at the Chebyshev nodes of [0, top]."""
    xs = [D(top) / 2 * (1 + D(math.cos(math.pi * (2 * i + 1) / (2 * terms)))) for i in range(terms)]
    a = [[x ** k for k in range(terms)] + [fn(x)] for x in xs]
    for i in range(terms):                     # Gauss-Jordan
        p = max(range(i, terms), key=lambda r: abs(a[r][i]))
        a[i], a[p] = a[p], a[i]
        a[i] = [v / a[i][i] for v in a[i]]
        for r in range(terms):
            if r != i:
                a[r] = [u - a[r][i] * v for u, v in zip(a[r], a[i])]
    return [row[-1] for row in a]


def poly(c, x):
    total = D(0)
    for v in reversed(c):
        total = total * x + v
    return total


def nearest(v):
    return float(Fraction(v))


def main():
    s_max = (D(2).sqrt() - 1) / (D(2).sqrt() + 1)
    z_max, t_max = s_max * s_max, D(1) / 16
    sets = (("kLog", q_exact, z_max, 7, lambda x, p: (2 + x * p) / (2 + x * q_exact(x)) - 1),
            ("kSin", s_exact, t_max, 6, lambda x, p: (PI + x * p) / (PI + x * s_exact(x)) - 1),
            ("kCos", c_exact, t_max, 7, lambda x, p: (1 + x * p) / (1 + x * c_exact(x)) - 1))
    for name, fn, top, terms, rel in sets:
        c = interpolate(fn, top, terms)
        worst = max(abs(rel(D(top) * i / 400, poly(c, D(top) * i / 400))) for i in range(401))
        print("constexpr double %s[%d] = {%s};" % (name, terms, ", ".join(nearest(v).hex() for v in c)))
        print("  // %.1e" % worst)


if __name__ == "__main__":
    main()
