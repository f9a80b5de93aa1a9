"""Makes the tables and coefficients of paper_1505_00965_amd/csrc/normal64.hpp.

Methods: the logarithm from a table of reciprocals 1/c and a polynomial in
r = z/c - 1 (P. T. P. Tang, Table-driven implementation of the logarithm
function in IEEE floating-point arithmetic, ACM TOMS 16, 1990); table points
searched so that the tabulated function values lie very near fp64 numbers (S.
Gal and B. Bachelis, An accurate elementary mathematical library for the IEEE
floating point standard, ACM TOMS 17, 1991); polynomials by interpolation at
Chebyshev nodes.  Everything is evaluated here in 60-digit decimals; numpy's
extended precision only narrows the searches.

Run it to print the constants in the header's form.
"""
import struct
from decimal import Decimal as D, getcontext

import numpy as np

getcontext().prec = 60
LOG_OFF, LOG_STEP, N = 0x3FE62000, 0x4000, 64


def pi():
    def atan_inv(n):
        s = t = D(1) / n
        k, sign = 1, -1
        while abs(t) > D(10) ** -62:
            t /= n * n
            k += 2
            s += sign * t / k
            sign = -sign
        return s
    return 4 * (4 * atan_inv(5) - atan_inv(239))


PI = pi()
LN2 = D(2).ln()


def sin_cos(x):
    """Taylor series after eight halvings."""
    x = x / 256
    s, c, ts, tc, k = x, D(1), x, D(1), 0
    while abs(tc) > D(10) ** -62:
        k += 2
        tc *= -x * x / (k * (k - 1))
        ts *= -x * x / (k * (k + 1))
        c += tc
        s += ts
    for _ in range(8):
        s, c = 2 * s * c, c * c - s * s
    return s, c


def nearest(x, scale):
    """x to the nearest multiple of 1 / scale."""
    return (x * scale).to_integral_value() / scale


def log_table():
    """[(1/c, -2 ln c)]: 1/c has 26 fractional bits, so that z/c - 1 is exact,
    and is, within 50000 of the interval's centre, the one whose -2 ln c is
    nearest to a multiple of 2^-47, to which it is rounded."""
    z = lambda hi: struct.unpack(">d", struct.pack(">Q", hi << 32))[0]
    out, rmax = [], 0.0
    for i in range(N):
        a, b = z(LOG_OFF + i * LOG_STEP), z(LOG_OFF + (i + 1) * LOG_STEP)
        if a < 1 < b:
            inv = 1.0
        else:
            mid = round(2 / (a + b) * 2 ** 26)
            k = np.arange(mid - 50000, mid + 50001)
            v = 2 * np.log(k.astype(np.longdouble) / 2 ** 26) * 2 ** 47
            inv = int(k[np.argmin(np.abs(v - np.rint(v)))]) / 2 ** 26
        rmax = max(rmax, abs(a * inv - 1), abs(b * inv - 1))
        out.append((inv, nearest(2 * D(inv).ln(), D(2 ** 47))))
    return out, rmax


def trig_table():
    """[(cos, sin, -d)] of 2 pi (i 2^26 + d) / 2^32: of d = 32, 64, ..., 5999 x 32
    the one whose cosine and sine lie nearest to fp64 values (d = 0 on the axes)."""
    out = []
    m = np.arange(1, 6000)
    w = np.longdouble(float(PI)) + np.longdouble(float(PI - D(float(PI))))
    for i in range(N):
        if i % 16 == 0:
            s, c = sin_cos(2 * PI * i / N)
            out.append((float(round(c)), float(round(s)), 0.0))
            continue
        # errors in units of 2^-53, good to 1e-3 in extended precision
        x = 2 * w * (i * 2 ** 26 + 32 * m).astype(np.longdouble) / np.longdouble(2) ** 32
        off = lambda v: np.abs(v - v.astype(np.float64).astype(np.longdouble)) * np.longdouble(2) ** 53
        e = np.maximum(off(np.cos(x)), off(np.sin(x)))
        best = None
        for k in m[e < e.min() + 5e-3]:
            s, c = sin_cos(2 * PI * (i * 2 ** 26 + 32 * int(k)) / 2 ** 32)
            err = max(abs(c - D(float(c))), abs(s - D(float(s))))
            if best is None or err < best[0]:
                best = (err, float(c), float(s), -32.0 * int(k))
        out.append(best[1:])
    return out


def chebyshev_fit(f, n, a, b):
    """Monomial coefficients of the interpolation of f at n Chebyshev nodes."""
    xs = [(a + b) / 2 + (b - a) / 2 * sin_cos(PI * (2 * k + 1) / (2 * n))[1] for k in range(n)]
    rows = [[x ** j for j in range(n)] + [f(x)] for x in xs]
    for i in range(n):                          # Gauss with pivots
        p = max(range(i, n), key=lambda r: abs(rows[r][i]))
        rows[i], rows[p] = rows[p], rows[i]
        for r in range(n):
            if r != i:
                q = rows[r][i] / rows[i][i]
                rows[r] = [u - q * v for u, v in zip(rows[r], rows[i])]
    return [float(rows[i][n] / rows[i][i]) for i in range(n)]


def polynomials(rmax):
    """(-2 ln(1 + r) + 2 r) / r^2 for |r| <= rmax; sin(w R) / R and
    (cos(w R) - 1) / R^2 in R^2 for |R| <= 2^25 + 1500 x 2^7, w = 2 pi / 2^32."""
    r = D(rmax)
    log = chebyshev_fit(lambda x: (-2 * (1 + x).ln() + 2 * x) / (x * x), 6, -r, r)
    top, w = D(2 ** 25 + 1500 * 2 ** 7), 2 * PI / 2 ** 32
    sin = chebyshev_fit(lambda y: sin_cos(w * y.sqrt())[0] / y.sqrt(), 4, D(0), top * top)
    cos = chebyshev_fit(lambda y: (sin_cos(w * y.sqrt())[1] - 1) / y, 4, D(0), top * top)
    return log, sin, cos


def constants():
    """Everything the header holds, by its names."""
    logs, rmax = log_table()
    hi = nearest(2 * LN2, D(2 ** 42))
    log, sin, cos = polynomials(rmax)
    return {"kLogTable": [(inv, float(25 * hi + l)) for inv, l in logs], "kTrigTable": trig_table(),
            "kLogPoly": log, "kSinPoly": sin, "kCosPoly": cos, "kTwoLn2Hi": float(hi), "kTwoLn2Lo": float(2 * LN2 - hi)}


def hex_of(v):
    return [hex_of(x) for x in v] if isinstance(v, (list, tuple)) else float(v).hex()


if __name__ == "__main__":
    for name, v in constants().items():
        print(name, "=")
        for row in (v if isinstance(v, list) else [v]):
            print("   ", hex_of(row))
