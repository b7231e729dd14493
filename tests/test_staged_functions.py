"""The functions the tiled and rows kernels evaluate for every pair, step by step on the host (Python doubles,
fused multiply-adds in exact rational arithmetic) against high-precision values: the exponential with the
biased table, the table logarithm, the series of ln(asin(s) / s), the angle halving of far pairs and the
sine behind it.  Constants and tables are read from the headers."""
import math
import os
import re
import struct
from decimal import Decimal, getcontext
from fractions import Fraction

import mpmath
import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2403_07412_amd", "csrc")
HEX = r"[-+]?0x[0-9a-fA-F.]+p[-+]?\d+"
getcontext().prec = 60


def _read(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def _pairs(name):
    return [(float.fromhex(a), float.fromhex(b)) for a, b in re.findall(r"\{(%s),\s*(%s)\}" % (HEX, HEX), _read(name))]


def _body(name, signature):
    text = _read(name)
    text = text[text.index(signature):]
    return text[:text.index("\n}\n")]


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _exp_constants():
    body = _body("device_common.h", "CovConst cov_const()")
    c = [float.fromhex(x) for x in re.findall(HEX, body)]
    return c  # eps, magic, -magic, -64 / ln2, -head, -tail


def test_exponential_constants():
    eps, magic, unmagic, inv, head, tail = _exp_constants()
    ln2_64 = Decimal(2).ln() / 64
    assert eps == 2.0 ** -1000 and magic == 1.5 * 2.0 ** 52 and unmagic == -magic
    assert abs(Decimal(-inv) - 1 / ln2_64) <= Decimal(math.ulp(inv)) / 2
    assert (math.frexp(-head)[0] * 2 ** 36).is_integer()  # n head is exact for |n| < 2^17
    assert abs(Decimal(-head) + Decimal(-tail) - ln2_64) < ln2_64 * Decimal(2) ** -90
    assert 708 * 64 / math.log(2) < 2 ** 17


@pytest.mark.parametrize("r", [0.0, 2.0 ** -500, 1e-9, 0.011, 0.5, 1.0, 7.25, 30.0, 333.3, 707.9, -0.3, -600.0])
def test_exponential_steps(r):
    _, magic, unmagic, inv, head, tail = _exp_constants()
    r = min(r, 708.0)
    t = fma(r, inv, magic)
    n = struct.unpack("<i", struct.pack("<d", t)[:4])[0]
    nf = t + unmagic
    assert nf == n
    f = fma(nf, tail, fma(nf, head, -r))
    a2 = (math.log(2) / 128) ** 2  # f^6 / 720 by its Chebyshev fit of lower degree
    q = fma(f, 1.0 / 120.0, 1.0 / 24.0 + 1.5 * a2 / 720.0)
    for c in (1.0 / 6.0, 0.5 - 0.5625 * a2 * a2 / 720.0, 1.0):
        q = fma(q, f, c)
    j = n & 63
    hi, lo = _pairs("exp_table.h")[j]
    bits = struct.unpack("<q", struct.pack("<d", hi))[0] + ((n - j) << 46)  # the high word plus (n - j) 2^14
    scaled = struct.unpack("<d", struct.pack("<q", bits))[0]
    got = fma(scaled, fma(q, f, lo / hi), scaled)
    exact = (-Decimal(r)).exp()
    assert abs(Decimal(got) - exact) <= Decimal(0.52) * Decimal(math.ulp(float(exact)))


def test_log_table():
    pairs = _pairs("log_table.h")
    assert len(pairs) == 64
    for j, (c, neg) in enumerate(pairs):
        lo, hi = 0.5 + j / 128, 0.5 + (j + 1) / 128
        assert (c * 1024).is_integer()
        assert abs(lo * c - 1) <= 2.0 ** -7 and abs(hi * c - 1) <= 2.0 ** -7
        exact = -Decimal(c).ln()
        assert abs(Decimal(neg) - exact) <= Decimal(math.ulp(neg)) / 2


@pytest.mark.parametrize("x", [1e-300, 3e-7, 0.4999, 0.99999999, 1.0, 1.0000001, 2.3, 1269.0, 4.1e8, 1e300])
def test_logarithm_steps(x):
    m, e = math.frexp(x)
    j = int((m - 0.5) * 128)
    c, neg = _pairs("log_table.h")[j]
    r = fma(m, c, -1.0)
    p = fma(r, 1.0 / 7.0, -1.0 / 6.0)
    for k in (1.0 / 5.0, -1.0 / 4.0, 1.0 / 3.0, -0.5):
        p = fma(p, r, k)
    p = fma(r * r, p, r)
    head, tail = float.fromhex("0x1.62e42fee00000p-1"), float.fromhex("0x1.a39ef35793c76p-33")
    got = fma(float(e), head, neg + fma(float(e), tail, p))
    exact = Decimal(x).ln()
    assert abs(Decimal(got) - exact) <= Decimal(0.75) * Decimal(math.ulp(float(exact))) + Decimal(2) ** -53


def test_log_of_arcsine_series():
    mpmath.mp.dps = 50
    body = _body("device_common.h", "__device__ __forceinline__ double pair_dist_pow(")
    body = body[body.index("double p = 36740617.0"):body.index("const double lnd")]
    coef = [Fraction(*map(int, f)) for f in re.findall(r"(\d+)\.0 / (\d+)\.0", body)]
    assert len(coef) == 7
    for h in (1e-12, 1e-4, 0.003, 0.01):
        H = mpmath.mpf(h)
        s = sum(mpmath.mpf(c.numerator) / c.denominator * H ** (7 - i) for i, c in enumerate(coef))
        exact = mpmath.log(mpmath.asin(mpmath.sqrt(H)) / mpmath.sqrt(H))
        assert abs(s - exact) < 1e-18


@pytest.mark.parametrize("h", [0.0100001, 0.05, 0.146, 0.5, 0.93, 0.9999999, 1.0])
def test_angle_halving(h):
    """asin sqrt h = 2^k asin sqrt h_k with h_k below 0.01 after at most four halvings, to a few ulps."""
    mpmath.mp.dps = 50
    x, k = h, 0
    while x > 0.01:
        x = (0.5 * x) / (1.0 + math.sqrt((1.0 - x) + 2.0 ** -1000))
        k += 1
    assert k <= 4
    exact = mpmath.asin(mpmath.sqrt(mpmath.mpf(h)))
    got = 2 ** k * mpmath.asin(mpmath.sqrt(mpmath.mpf(x)))
    assert abs(got / exact - 1) < 4 * 2.0 ** -53


def test_quarter_sine():
    mpmath.mp.dps = 50
    body = _body("device_common.h", "__device__ __forceinline__ double sin_quarter(")
    coef = [s * 1.0 / float(n) for s, n in ((-1.0 if m else 1.0, int(n)) for m, n in
            re.findall(r"(-)?1\.0 / (\d+)\.0", body))]
    assert len(coef) == 8
    for x in np.linspace(1e-6, math.pi / 4, 60):
        x = float(x)
        z = x * x
        q = coef[0]
        for c in coef[1:]:
            q = fma(q, z, c)
        got = fma(x * z, q, x)
        exact = mpmath.sin(mpmath.mpf(x))
        assert abs(got - exact) <= 0.75 * math.ulp(float(exact))
