"""The device logarithm (csrc/device/math.hip, ln) on the host: its sequence of
operations, emulated with exactly rounded FMAs and the coefficients read from
the source, against 40-digit logarithms.  No GPU.

Tolerance: 2 ulp.  The reduced logarithm u = s2 + s2 z q carries at most 1 ulp
of itself (the rounded quotient's correction and the last FMA's half ulp), the
two FMAs that add e ln 2 half an ulp of the result each; |u| is at most that of
the result unless they cancel, and they cannot: e is 0 for arguments in
[0.7, 1.41)."""
import decimal
import math
import pathlib
import re
import struct
from fractions import Fraction

import numpy as np
import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
SRC = (ROOT / "paper_2508_16105_amd" / "csrc" / "device" / "math.hip").read_text()


def _coefficients():
    i = SRC.index("double ln(double x)")
    body = SRC[i:SRC.index("\n}\n", i)]
    first = re.search(r"double q = fma\(([-+0-9.e]+), z, ([-+0-9.e]+)\);", body)
    return [float(first.group(1)), float(first.group(2))] + [
        float(c) for c in re.findall(r"q = fma\(q, z, ([-+0-9.e]+)\);", body)]


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _ln(x, co):
    bits = struct.unpack("<q", struct.pack("<d", x))[0]
    e = (bits - 0x3FE6A09E00000000) >> 52
    m = struct.unpack("<d", struct.pack("<q", bits - (e << 52)))[0]
    f, d = m - 1.0, m + 1.0
    r = 1.0 / d
    s = f * r
    s = _fma(r, _fma(-s, d, f), s)
    z = s * s
    q = _fma(co[0], z, co[1])
    for c in co[2:]:
        q = _fma(q, z, c)
    s2 = s + s
    u = _fma(s2, z * q, s2)
    return _fma(float(e), 0.6931471805599453, _fma(float(e), 2.3190468138462996e-17, u))


@pytest.mark.parametrize("lo,hi", [(0.70710678, 1.41421357), (200.0, 6000.0), (1e-300, 1e300)])
def test_ln_within_two_ulp(lo, hi):
    co = _coefficients()
    rng = np.random.default_rng(7)
    x = np.concatenate([np.exp(rng.uniform(math.log(lo), math.log(hi), 1500)), [lo, hi]])
    if lo < 1.0 < hi:
        x = np.concatenate([x, 1.0 + rng.uniform(-1e-6, 1e-6, 200), [1.0, np.nextafter(1.0, 0), np.nextafter(1.0, 2)]])
    with decimal.localcontext() as ctx:
        ctx.prec = 40
        for v in map(float, x):
            ref = decimal.Decimal(v).ln()
            y = _ln(v, co)
            if v == 1.0:
                assert y == 0.0
                continue
            assert abs(decimal.Decimal(y) - ref) <= 2 * decimal.Decimal(math.ulp(float(ref))), v
