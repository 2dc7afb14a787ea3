"""The quotient by a reciprocal that the TLI row pass evaluates (csrc/tli.hip: quotient), in exact rational
arithmetic: the IEEE nearest fp32 quotient over the range in which the kernel uses it."""
from fractions import Fraction

import numpy as np


def rn(x):
    """The nearest fp32 to a rational in the normal range, ties to even."""
    if x == 0:
        return Fraction(0)
    sign, x = (1, x) if x > 0 else (-1, -x)
    e = x.numerator.bit_length() - x.denominator.bit_length()
    e -= 1 if Fraction(2) ** e > x else 0
    unit = Fraction(2) ** (e - 23)
    q = x / unit
    f, rem = q.numerator // q.denominator, q - q.numerator // q.denominator
    f += 1 if rem > Fraction(1, 2) or (rem == Fraction(1, 2) and f % 2) else 0
    return sign * f * unit


def quotient(g, S):
    r = rn(1 / S)
    q0 = rn(g * r)
    q1 = rn(q0 + rn(g - q0 * S) * r)
    return rn(q1 + rn(g - q1 * S) * r)


def test_quotient_is_the_nearest():
    rng = np.random.default_rng(81)
    lo, hi = (int(np.float32(v).view(np.uint32)) for v in (2.0 ** -30, 2.0 ** 10))
    g_lo = int(np.float32(2.0 ** -60).view(np.uint32))
    for i in range(6000):
        S = int(rng.integers(lo, hi + 1))
        if i % 3 == 1:
            S |= 0x7FFFFF - int(rng.integers(0, 4))  # mantissas near all ones
        elif i % 3 == 2:
            S = int(np.float32(1.0 - 2.0 ** -24 * int(rng.integers(0, 64))).view(np.uint32))  # masses near one
        g = int(rng.integers(g_lo, 0x3F800000 + 1)) if i % 2 else int(np.float32(rng.random()).view(np.uint32))
        if S > hi or g < g_lo:
            continue
        Sf, gf = (Fraction(float(np.uint32(v).view(np.float32))) for v in (S, g))
        assert quotient(gf, Sf) == rn(gf / Sf), (hex(g), hex(S))
