"""The FP32 distance of a sphere about the origin is the square root of an
operand known to the bit, less the radius: fma(x, x, fl(y y)) at a point
(x, y, 0).  One rounding each, so every result is equal to the host's."""
import math
from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _f32(v):
    """the FP32 nearest to a fraction v >= 0 (ties to even, denormals kept)"""
    if v == 0:
        return np.float32(0.0)
    e = v.numerator.bit_length() - v.denominator.bit_length()
    e -= Fraction(2) ** e > v
    q = max(e - 23, -149)
    return np.float32(math.ldexp(round(v / Fraction(2) ** q), q))


def _operands(x, y):
    yy = y * y
    return np.array([_f32(Fraction(float(a)) ** 2 + Fraction(float(b))) for a, b in zip(x, yy)], dtype=np.float32)


def _check(S, W, eng, x, y, r):
    desc = W.absorbing_sphere(r=float(np.float32(r)))
    desc["delta"] = float(r) * 1e-3
    desc["pad"] = float(r) * 1e-2
    pts = np.zeros((x.size, 3))
    pts[:, 0], pts[:, 1] = x, y
    d, _ = S.distance(desc, pts, engine=eng, precision="f32")
    want = np.sqrt(_operands(x, y)) - np.float32(r)
    bad = np.nonzero(d[:, 0].astype(np.float32) != want)[0]
    assert bad.size == 0, (bad.size, [(float(x[i]), float(y[i]), d[i, 0], float(want[i])) for i in bad[:4]])


@pytest.mark.parametrize("size", [1.0, 3e4, 1e-6, 2.0 ** -45])
def test_roots_next_to_midpoints(S, W, eng, size):
    """operands as near as FP32 has them to the square of a number half way
    between two neighbours, where the last bit of the root is decided"""
    g = np.random.default_rng(7)
    s = (size * g.uniform(0.5, 2.0, 6000)).astype(np.float32)
    mid = s.astype(np.float64) + 0.5 * np.spacing(s).astype(np.float64)
    y = np.sqrt(mid * mid - s.astype(np.float64) ** 2).astype(np.float32)
    near = [y, np.nextafter(y, np.float32(0)), np.nextafter(y, np.float32(np.inf))]
    _check(S, W, eng, np.concatenate([s] * 3), np.concatenate(near), size * 2.0 ** -20)


@pytest.mark.parametrize("lo,hi", [(2.0 ** -49, 2.0 ** -47), (1e-18, 1e-14), (2.0 ** -64, 2.0 ** -62), (1e-23, 1e-19)])
def test_small_lengths_are_correctly_rounded(S, W, eng, lo, hi):
    """lengths about 2^-48, below it, and where the operand is denormal or 0"""
    g = np.random.default_rng(8)
    x, y = (np.exp(g.uniform(math.log(lo), math.log(hi), 4000)).astype(np.float32) for _ in range(2))
    y[::3] = 0.0
    x[0] = 0.0
    _check(S, W, eng, x, y, lo * 2.0 ** -8)
