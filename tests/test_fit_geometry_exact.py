"""The extrapolation's scan window of half-width 2 with power-of-two weights:
the HIP fit counts its normal matrix from the 25-bit mask of the valid nodes
and keeps cofactors and determinant as integers.  The same counts here against
exact rational sums, with the bounds that the 24-bit products and the packed
fields need, and the claim that 4096 / det rounded to float does not depend on
the last place of the double quotient."""
from fractions import Fraction

import numpy as np

NODES = [(a, b) for b in range(-2, 3) for a in range(-2, 3)]


def _count(mask, f):
    return sum(1 for k, (a, b) in enumerate(NODES) if (a or b) and mask >> k & 1 and f(a, b))


def _geometry(mask):
    n = lambda f: _count(mask, f)  # noqa: E731
    m22 = sum(w * n(lambda a, b, d=d: abs(a) + abs(b) == d) for d, w in ((1, 8), (2, 4), (3, 2), (4, 1)))
    m02 = sum(w * (n(lambda a, b: a > 0 and abs(b) == k) - n(lambda a, b: a < 0 and abs(b) == k))
              for k, w in ((0, 8), (1, 4), (2, 2)))
    m12 = sum(w * (n(lambda a, b: b > 0 and abs(a) == k) - n(lambda a, b: b < 0 and abs(a) == k))
              for k, w in ((0, 8), (1, 4), (2, 2)))
    m00 = sum(8 * abs(a) >> abs(b) for k, (a, b) in enumerate(NODES) if mask >> k & 1 and (a or b))
    m11 = sum(8 * abs(b) >> abs(a) for k, (a, b) in enumerate(NODES) if mask >> k & 1 and (a or b))
    m01 = 4 * (n(lambda a, b: a * b > 0) - n(lambda a, b: a * b < 0))
    return m00, m01, m02, m11, m12, m22


def test_normal_matrix_from_the_validity_mask_is_exact():
    rng = np.random.default_rng(1)
    masks = [0, (1 << 25) - 1 - (1 << 12)] + [int(m) & ~(1 << 12) for m in
                                              rng.integers(0, 1 << 25, 3000)]
    for mask in masks:
        m = _geometry(mask)
        w = [(Fraction(1, 2 ** (abs(a) + abs(b))), a, b) for k, (a, b) in enumerate(NODES)
             if mask >> k & 1]
        exact = [sum(q * a * a for q, a, b in w), sum(q * a * b for q, a, b in w),
                 sum(q * a for q, a, b in w), sum(q * b * b for q, a, b in w),
                 sum(q * b for q, a, b in w), sum(q for q, a, b in w)]
        assert [Fraction(v, 16) for v in m] == exact
        m00, m01, m02, m11, m12, m22 = m
        # the records' fields: unsigned and signed bytes
        assert 0 <= m00 < 256 and 0 <= m11 < 256
        assert all(-128 <= v < 128 for v in (m01, m02, m12))
        c = (m01 * m12 - m11 * m02, m01 * m02 - m00 * m12, m00 * m11 - m01 * m01)
        assert all(abs(v) < 1 << 23 for v in c)
        det = m02 * c[0] + m12 * c[1] + m22 * c[2]
        assert 0 <= det < 1 << 21


def test_rounded_reciprocal_of_the_determinant_is_unique():
    # the quotient in double and its neighbours round to the same float
    # (512 / det, as the FP32 fit takes it; powers of two are exact)
    d = np.arange(1, 1 << 21, dtype=np.float64)
    q = 512.0 / d
    keep = np.log2(d) % 1 != 0
    f = q.astype(np.float32)
    assert np.array_equal(f[keep], np.nextafter(q, np.inf).astype(np.float32)[keep])
    assert np.array_equal(f[keep], np.nextafter(q, -np.inf).astype(np.float32)[keep])
