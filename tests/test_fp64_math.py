"""The march's own FP64 reciprocal, quotient, square root and logarithm, function by function, from
seeds cut to 24 fraction bits (a little coarser than the hardware's), against extended precision.

Bounds, in units of eps = 2^-53 of the value, with a seed error of at most 2^-24:
  1/x       seed error cubed (2^-72) and the rounding of e + e^2 times r (2^-24 eps) vanish beside
            the last rounding: 1 and a bit;
  x/y       the quotient is corrected by its own remainder: 1 and a bit;
  sqrt x    the same;
  x + y/z   the last rounding (1 of the sum) and 1 and a bit of y/z;
  1/x of the three: the seed error squared (2^-48 = 32 eps) and six products.
"""
import mpmath as mp
import numpy as np
import pytest

import emulator as EM

EPS = 2.0 ** -53
N = 4000


def _wide(seed, lo, hi, n=N):
    """Log-uniform arguments, with the ends and the neighbours of powers of two among them."""
    rng = np.random.default_rng(seed)
    x = np.exp2(rng.uniform(np.log2(lo), np.log2(hi), n))
    p = np.exp2(np.arange(np.ceil(np.log2(lo)), np.floor(np.log2(hi)) + 1))
    return np.clip(np.concatenate([x, p, np.nextafter(p, 0), np.nextafter(p, np.inf), [lo, hi]]), lo, hi)


def _errors(got, exact):
    """|got - exact| / |exact| in eps; exact(k) in extended precision."""
    mp.mp.prec = 160
    return np.array([float(abs(mp.mpf(float(g)) / exact(k) - 1) / EPS) for k, g in enumerate(got)])


def test_reciprocal():
    x = _wide(1, 4.0, 1e300)
    assert _errors(EM.fp64_math(0, x), lambda k: 1 / mp.mpf(float(x[k]))).max() <= 1.01


def test_quotient():
    y = _wide(2, 0.04, 1e150)
    x = np.random.default_rng(3).normal(size=y.size) * 10.0
    x[0], x[1] = 1.0, -3.0
    assert _errors(EM.fp64_math(1, x, y), lambda k: mp.mpf(float(x[k])) / mp.mpf(float(y[k]))).max() <= 1.01


def test_square_root():
    x = _wide(4, 1.0, 1e150)
    assert _errors(EM.fp64_math(2, x), lambda k: mp.sqrt(mp.mpf(float(x[k])))).max() <= 1.01


def test_sum_with_a_quotient():
    z = _wide(5, 1e3, 1e150)
    rng = np.random.default_rng(6)
    x, y = rng.normal(size=z.size), rng.normal(size=z.size) * z
    mp.mp.prec = 160
    got = EM.fp64_math(5, x, y, z)
    for k in range(z.size):
        q = mp.mpf(float(y[k])) / mp.mpf(float(z[k]))
        s = mp.mpf(float(x[k])) + q
        assert abs(mp.mpf(float(got[k])) - s) <= EPS * (abs(s) + 1.01 * abs(q))


def test_three_reciprocals():
    rng = np.random.default_rng(7)
    q = 4.0 + np.exp2(rng.uniform(-20, 60, (N, 3)))
    got = EM.fp64_math(4, *q.T.copy())
    for c in range(3):
        err = _errors(got[:, c], lambda k: 1 / mp.mpf(float(q[k, c])))
        assert err.max() <= 32 + 6.5


@pytest.mark.parametrize("lo,hi", [(1.0, 1.001), (1.0, 2.0), (1.0, 64.0), (1.0, 1e150)])
def test_logarithm(lo, hi):
    x = _wide(8, lo, hi)
    x = x[x > 1.0]
    got = EM.fp64_math(3, x)
    err = _errors(got, lambda k: mp.log(mp.mpf(float(x[k]))))
    assert EM.fp64_math(3, np.array([1.0]))[0] == 0.0
    print("largest %.3f, rms %.3f eps" % (err.max(), np.sqrt((err ** 2).mean())))
    assert err.max() <= 4.0


@pytest.mark.parametrize("lo,hi", [(1.0, 1.1), (1.0, 1.5), (1.3, 3.0), (1.0, 1e150)])
def test_logarithm_rounds_once(lo, hi):
    """ln is the rounded sum of a head and its remainder.  What is not in either: of s (d^2/2 + z Q),
    at most d^2/2 times half of |ln m|, the 5 roundings of its factors and the products' two; of
    the remainder sums one rounding each of terms below 2^-52 of ln; for |d| <= 0.415 that is
    under 7 * 0.043 + 0.01 of eps, with the last rounding 1.31 (and it was up to 2.8)."""
    rng = np.random.default_rng(9)
    x = np.exp2(rng.uniform(np.log2(lo), np.log2(hi), 3 * N))
    x = x[x > 1.0]
    err = _errors(EM.fp64_math(3, x), lambda k: mp.log(mp.mpf(float(x[k]))))
    print("largest %.3f, rms %.3f eps" % (err.max(), np.sqrt((err ** 2).mean())))
    assert err.max() <= 1.31
