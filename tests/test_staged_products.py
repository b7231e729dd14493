"""The covariance and its beta-derivative at scaled distances past the range of the exponential, on the host:
the steps of the staged exponential with the header's clamp, times the powers of the clamped distance that the
closed forms multiply it by."""
import math
import random
import re
import struct
from decimal import Decimal, getcontext

import pytest

from test_staged_functions import _body, _exp_constants, _pairs, _read, fma


def _clamp():
    return float(re.findall(r"[\d.]+", _body("device_common.h", "CovConst cov_const()").split("}")[0])[-1])


def _exp_neg(r):
    _, magic, unmagic, inv, head, tail = _exp_constants()
    t = fma(r, inv, magic)
    n = struct.unpack("<i", struct.pack("<d", t)[:4])[0]
    nf = t + unmagic
    f = fma(nf, tail, fma(nf, head, -r))
    hi, lo = _pairs("exp_table.h")[n & 63]
    return math.ldexp(fma(hi, math.expm1(f) + lo / hi, hi), n >> 6)


@pytest.mark.parametrize("beta", [1e-3, 7.5e-4, 6.95e-4, 6.8e-4, 1e-6, 1e-78, 1e-103, 1e-160, 1e-300])
def test_products_vanish_with_the_exponential(beta):
    r = min(0.5 / beta, _clamp())
    e = _exp_neg(r)
    for power in (1, 2, 3):
        got = r ** power * e
        exact = Decimal(0.5 / beta) ** power * (-Decimal(0.5 / beta)).exp()
        assert abs(Decimal(got) - exact) <= Decimal(1e-15) * exact + Decimal(5e-324) * Decimal(r) ** power


def test_clamp_is_the_first_zero():
    c = _clamp()
    assert _exp_neg(c) == 0.0 and 0.0 < _exp_neg(c - 2.0) < 1e-322


def _staged_exp(r):
    """exp_neg_staged's own lines and constants, statement by statement."""
    text = _body("device_common.h", "struct CovConst {")
    names = [x.strip() for line in re.findall(r"double ([^;]+);", text) for x in line.split(",")]
    init = _body("device_common.h", "CovConst cov_const()")
    values = re.search(r"CovConst c\{(.*?)\};", init, re.S).group(1).split(",")
    a2 = re.search(r"constexpr double A2 = (.*?);", init)
    scope = {"A2": eval(a2.group(1))} if a2 else {}

    def number(x):
        return re.sub(r"-?0x[0-9a-f.]+p[-+]?\d+", lambda h: repr(float.fromhex(h.group(0))), x.strip())

    const = {n: eval(number(v), scope) for n, v in zip(names, values)}
    body = _body("device_common.h", "__device__ __forceinline__ double exp_neg_staged(")
    t = fma(r, const["inv_ln2_64"], const["magic"])
    env = {"fma": fma, "c": type("C", (), const), "r": r, "t": t, "nf": t + const["unmagic"]}
    n = struct.unpack("<i", struct.pack("<d", t)[:4])[0]
    for var, expr in re.findall(r"\b([fq]) = (fma\([^;]*\));", body):
        env[var] = eval(expr, env)
    hi, lo = _pairs("exp_table.h")[n & 63]
    return math.ldexp(fma(hi, fma(env["q"], env["f"], lo / hi), hi), n >> 6)


def test_exponential_rounds_once():
    """Half an ulp for the last rounding; 0.004 for the correction's (below 2^-7.5, rounded to 53 bits), 0.003
    for the polynomial's, and the truncated f^7 / 5040: 0.508 ulp, the bound of the unstaged form as well."""
    rng = random.Random(5)
    getcontext().prec = 40
    for _ in range(3000):
        r = rng.uniform(0.0, 40.0)
        exact = (-Decimal(r)).exp()
        ulp = Decimal(2) ** (math.frexp(float(exact))[1] - 53)
        assert abs(Decimal(_staged_exp(r)) - exact) <= Decimal("0.508") * ulp, r


def test_logarithm_near_one():
    """Within 2^-8 of 1 the table's term is below 2^-6 and its rounding and that of the sum with it below 2^-59
    each; the result's own rounding is smaller."""
    text = _read("log_table.h")
    low = [float.fromhex(x) for x in re.findall(r"0x[\d.a-f]+p[-+]\d+", text[text.index("kLogMantLow["):].split("}")[0])]
    pairs = _pairs("log_table.h")
    getcontext().prec = 40
    for (c, _), neg in zip(pairs, low):
        exact = -(Decimal(c) / 2).ln()
        assert abs(Decimal(neg) - exact) <= Decimal(math.ulp(neg)) / 2
    head, tail = float.fromhex("0x1.62e42fee00000p-1"), float.fromhex("0x1.a39ef35793c76p-33")
    rng = random.Random(9)
    for x in [1.0, 1.0 + 2.0 ** -52, 1.0 - 2.0 ** -53] + [1.0 + rng.uniform(-2.0 ** -8, 2.0 ** -8) for _ in range(2000)]:
        m, e = math.frexp(x)
        j = int((m - 0.5) * 128)
        c, neg = pairs[j]
        if j < len(low):
            e, neg = e - 1, low[j]
        r = fma(m, c, -1.0)
        p = fma(r, 1.0 / 7.0, -1.0 / 6.0)
        for k in (1.0 / 5.0, -1.0 / 4.0, 1.0 / 3.0, -0.5):
            p = fma(p, r, k)
        got = fma(float(e), head, neg + fma(float(e), tail, fma(r * r, p, r)))
        assert abs(Decimal(got) - Decimal(x).ln()) <= Decimal(2) ** -58, x
