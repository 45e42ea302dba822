"""The products that the split GEMMs form (MKOR_GEMM_SPLIT), checked on the CPU
against float64: a row's scaled fp16 pairs x = h + l, the three partial
products kept, the fourth left out, and the one plane of a bf16 gradient."""
import numpy as np

from oracle.half import round_bf16
from tests.test_split_scale import pair, split_exp


def _row(rng, n, emin, emax):
    """n values of magnitudes from 2^emin to 2^emax, as one row."""
    return (rng.choice([-1.0, 1.0], n) * np.ldexp(rng.uniform(1.0, 2.0, n), rng.integers(emin, emax, n))).astype(np.float32)


def test_kept_products_are_exact_in_fp32():
    """Every factor has 11 significant bits: 22 in a product."""
    rng = np.random.default_rng(0)
    (hx, lx), (hy, ly) = pair(_row(rng, 100_000, -14, 0)), pair(_row(rng, 100_000, -14, 0))
    for p in (hx * hy, hx * ly, lx * hy):
        assert np.array_equal(p, p.astype(np.float32).astype(np.float64))


def test_dropped_product_is_below_fp32_rounding():
    """Where no entry falls under fp16's spacing, |l l'| <= 2^-22 |x x'|, and the
    kept three are within 2^-21 |x x'| of the product."""
    rng = np.random.default_rng(1)
    x, y = _row(rng, 100_000, -14, 0), _row(rng, 100_000, -14, 0)
    (hx, lx), (hy, ly) = pair(x), pair(y)
    xy = x.astype(np.float64) * y.astype(np.float64)
    assert np.all(np.abs(lx * ly) <= 2.0 ** -22 * np.abs(xy))
    assert np.all(np.abs(hx * hy + hx * ly + lx * hy - xy) <= 2.0 ** -21 * np.abs(xy))


def test_bf16_gradient_is_one_exact_plane():
    """Down to 2^-31 of the row's largest entry; below, bits are lost, and below
    2^-40 the value."""
    rng = np.random.default_rng(2)
    g = round_bf16(np.ldexp(rng.uniform(1.0, 2.0, 100_000), rng.integers(-30, 1, 100_000)))
    s = np.ldexp(g, split_exp(g.max()))
    assert np.array_equal(s.astype(np.float16).astype(np.float64), s)
    e = split_exp(1.0)
    low = round_bf16([2.0 ** -33 * (1 + 2.0 ** -7)])
    assert np.ldexp(low, e).astype(np.float16).astype(np.float64) != np.ldexp(low, e)
    assert np.ldexp(round_bf16([2.0 ** -41]), e).astype(np.float16) == 0


def test_split_limits():
    """Scales stop at 2^126, so rows of subnormal numbers keep what fp16 holds;
    rows of the largest finite ones do not overflow; a row with an infinity has
    the scale 1."""
    assert split_exp(np.float32(2.0 ** -140)) == 126 and split_exp(np.float32(0.0)) == 0
    assert split_exp(np.float32(np.inf)) == 0
    x = np.float32([3.4e38, -3.4e38, 1e30])
    h, l = pair(x)
    assert np.all(np.abs(h + l - x.astype(np.float64)) <= 2.0 ** -23 * np.abs(x) + 2.0 ** -39 * 3.4e38)
