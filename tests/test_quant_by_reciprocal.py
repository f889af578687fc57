"""The quantisation kernels form x / s as t = x * fl(1 / s), corrected once: fl(t + fl(x - t s) * fl(1 / s))
with fused multiply-adds.  For s = fl(amax / 127) of a bf16 maximum that is the binary32 quotient to the
bit, over every pair of significands: checked here in exact arithmetic.  (Powers of two change nothing
as long as nothing underflows; quotients below 2^-5 round to zero either way.)"""
from fractions import Fraction

import numpy as np


def round32(v):
    """A fraction rounded to a significand of 24 bits, half to even."""
    if v == 0:
        return Fraction(0)
    a, unit = abs(v), Fraction(1)
    while a >= 2 ** 24 * unit:
        unit *= 2
    while a < 2 ** 23 * unit:
        unit /= 2
    n = round(a / unit)  # (half to even)
    return n * unit if v > 0 else -n * unit


def test_corrected_products_are_the_quotients():
    f32 = np.float32
    significands = (1 + np.arange(128) / 128).astype(f32)
    s = significands / f32(127)
    products = 0
    for sv, inv in zip(s, f32(1) / s):
        S, I = Fraction(float(sv)), Fraction(float(inv))
        for x in significands:
            want, t = x / sv, x * inv
            X, T = Fraction(float(x)), Fraction(float(t))
            assert round32(T + round32(X - T * S) * I) == Fraction(float(want)), (sv, x)
            products += want == t
    assert 0 < products < 128 * 128  # (the products alone are not the quotients)
