"""The histogram's quotient without a division: q = RN(g inv), r = g - q a exactly, then
RN(q + r inv), inv = RN(1 / a), equals RN(g / a) for every pair of float32 values |g| <= a.
The same steps in exact rational arithmetic (float(Fraction) rounds to nearest even),
against the division, on the pairs where it could go wrong: mantissas at both ends of a
binade, neighbours, exact quotients, subnormals, and random ones.
"""
import random
import struct
from fractions import Fraction

import pytest


def _f32(bits):
    return struct.unpack("<f", struct.pack("<I", bits))[0]


def _fma(x, y, z):
    return float(Fraction(x) * Fraction(y) + Fraction(z))


def _quotient(g, a):
    inv = 1.0 / a
    q = g * inv
    return _fma(_fma(-q, a, g), inv, q)


def _pairs(kind, rng):
    top = 0x7F7FFFFF
    for _ in range(4000):
        if kind == "random":
            a, g = rng.randint(1, top), rng.randint(0, top)
        elif kind == "binade_ends":
            e = rng.randint(1, 254) << 23
            a = e | rng.choice([0, 1, 2, 0x7FFFFF, 0x7FFFFE, rng.getrandbits(23)])
            g = max(0, a - (rng.randint(0, 30) << 23)) & ~0x7FFFFF | rng.choice(
                [0, 1, 0x7FFFFF, 0x7FFFFE, rng.getrandbits(23)])
        elif kind == "neighbours":
            a = rng.randint(64, top)
            g = a - rng.randint(0, 63)
        elif kind == "bf16":
            a, g = rng.randint(1, 0x7F7F) << 16, rng.randint(0, 0x7F7F) << 16
        else:   # subnormals, and the smallest over the largest
            a = rng.choice([rng.randint(1, 0x7FFFFF), top, 0x00800000])
            g = rng.randint(0, min(a, 0x7FFFFF))
        a, g = _f32(a), _f32(g)
        yield min(g, a), max(g, a)


@pytest.mark.parametrize("kind", ["random", "binade_ends", "neighbours", "bf16", "subnormal"])
def test_quotient_is_the_rounded_division(kind):
    rng = random.Random(7)
    for g, a in _pairs(kind, rng):
        if a == 0.0:
            continue
        for s in (g, -g):
            assert _quotient(s, a) == s / a, (s.hex(), a.hex())
