"""The sampler skips the Gumbel variate of an entry whose score cannot win.  It decides that from
bounds on the variate by the logarithm of the uniform's complement; a bound that
failed for some random word would silently drop a winner once in a long while, which random parity
runs need not catch.  Here the bounds are checked for every value the uniform can take (the variate
depends on the upper 23 bits of a random word), against the Gumbel transform in float64 and, on a
sample, against the oracle's binary32 routine."""
import numpy as np

import oracle


def _bounds_from_x(k):
    """k = the 23 bits of a random word that make the uniform u = (2 k + 1) 2^-24.  The bounds the kernel uses, in its
    own binary32 operations but for the logarithm, which is rounded from float64: x = 1 - u, G <= -ln x + 1e-3 and
    G >= -ln x - 2.82 x - 1e-3."""
    f = np.float32
    x = (f(1) - f(2.0 ** -24)) - k.astype(f) * f(2.0 ** -23)          # exact: see the test
    neg_ln = -(np.log2(x.astype(np.float64)).astype(f).astype(np.float64) * float(f(0.69314718)))
    return x, neg_ln - 2.82 * x.astype(np.float64) - 1e-3, neg_ln + 1e-3


def test_bounds_hold_for_every_uniform():
    k = np.arange(1 << 23, dtype=np.int64)
    x, lower, upper = _bounds_from_x(k)
    m = (0x00FFFFFF ^ (k << 1)).astype(np.int64)                       # (1 - u) 2^24: odd, 1 .. 2^24 - 1
    assert m.min() == 1 and m.max() == (1 << 24) - 1 and (m & 1).all()
    assert (x.astype(np.float64) * 2.0 ** 24 == m).all(), "the complement is exact"
    g = -np.log(-np.log((2 * k + 1).astype(np.float64) * 2.0 ** -24))
    # 9e-4 of the margin are left for the hardware logarithm (1e-6 of at most 17) and the variate's routine (1e-6)
    assert (g <= upper - 9e-4).all(), "upper bound"
    assert (g >= lower + 9e-4).all(), "lower bound"
    # for the large variates that win they are close: within 3 x + 2e-3
    assert np.all(upper - lower <= 2.82 * x.astype(np.float64) + 2.1e-3)


def test_bounds_hold_for_the_binary32_routine():
    oracle.build()
    rng = np.random.default_rng(11)
    ks = np.concatenate([rng.integers(0, 1 << 23, 20000), np.arange(0, 4096), (1 << 23) - 1 - np.arange(0, 4096),
                         (1 << np.arange(0, 23)), (1 << np.arange(1, 23)) - 1]).astype(np.int64)
    _, lower, upper = _bounds_from_x(ks)
    low_bits = rng.integers(0, 512, ks.size)
    for k, lb, lo, up in zip(ks, low_bits, lower, upper):
        g = oracle.gumbel(int((k << 9) | lb))   # the lower 9 bits of the word do not matter
        # (9e-4: as above)
        assert lo + 9e-4 <= g <= up - 9e-4, (k, g, lo, up)
