"""The binary32 determinant, U, W and T of a pair have one value in every kernel: the
grouping into fused operations is written out, not left to each kernel's
compilation.  Against that grouping in exact rational arithmetic, each operation
rounded once to the nearest."""
from fractions import Fraction

import numpy as np
import pytest

import paper_2305_01867_amd as rsi
from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


def _round(x):
    """The binary32 value nearest to a rational, ties to the even one."""
    c = np.float32(float(x))
    near = [np.nextafter(c, np.float32(-np.inf)), c, np.nextafter(c, np.float32(np.inf))]
    return min(near, key=lambda v: (abs(Fraction(float(v)) - x), int(v.view(np.uint32)) & 1))


def _mul(a, b):
    return _round(Fraction(float(a)) * Fraction(float(b)))


def _fma(a, b, c):
    return _round(Fraction(float(a)) * Fraction(float(b)) + Fraction(float(c)))


def _cross(a, b):
    return [_fma(a[i], b[j], -_mul(a[j], b[i])) for i, j in ((1, 2), (2, 0), (0, 1))]


def _dot(a, b):
    return _fma(a[2], b[2], _fma(a[0], b[0], _mul(a[1], b[1])))


def test_the_quantities_of_a_pair_follow_the_written_grouping():
    rng = np.random.default_rng(11)
    n = 400
    O, E = (rng.uniform(-1, 1, (n, 3)).astype(np.float32) for _ in range(2))
    C = rng.uniform(-1, 1, (n, 3, 3)).astype(np.float32)
    vals = host(rsi.rsi_debug_certify(dev(O), dev(E), dev(C))[0])
    for k in range(n):
        d, a, e1, e2 = E[k] - O[k], C[k, 0], C[k, 1] - C[k, 0], C[k, 2] - C[k, 0]
        s = O[k] - a
        p, q = _cross(d, e2), _cross(s, e1)
        want = np.array([_dot(e1, p), _dot(s, p), _dot(d, q), _dot(e2, q)], np.float32)
        assert np.array_equal(vals[k, :4].view(np.uint32), want.view(np.uint32)), k
