"""The covariance and its beta-derivative at scaled distances past the range of the exponential, on the host:
the steps of the staged exponential with the header's clamp, times the powers of the clamped distance that the
closed forms multiply it by."""
import math
import re
import struct
from decimal import Decimal

import pytest

from test_staged_functions import _body, _exp_constants, _pairs, fma


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
