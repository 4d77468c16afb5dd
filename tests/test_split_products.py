"""The arithmetic behind the float32 path's matrix products, on the CPU: a float32 value as three bfloat16 parts, six of the nine products of two
such sums, and what each of the six is worth to a sum (the bounds of test_gpu_f32_split.py lie between)."""
import numpy as np
import pytest


def _bf16(x):
    """float32 -> bfloat16 to nearest even, as float32"""
    u = x.astype(np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & np.uint32(0xFFFF0000)).view(np.float32)


def _parts(x, scale=np.float32(2.0 ** 24)):
    x = x.astype(np.float32) * scale
    h = _bf16(x)
    m = _bf16(x - h)
    return [p.astype(np.float64) / float(scale) for p in (h, m, _bf16(x - h - m))]


KEPT = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]


def _products(x, y, kept=KEPT):
    px, py = _parts(x), _parts(y)
    return sum(px[i] * py[j] for i, j in kept)


@pytest.mark.parametrize("exponent", [-149, -126, -110, 0, 100])
def test_three_parts_are_the_value(exponent):
    x = np.ldexp(np.random.default_rng(1).uniform(1, 2, 4096), exponent).astype(np.float32)
    np.testing.assert_array_equal(sum(_parts(x)), x.astype(np.float64))


def test_parts_without_the_factor_lose_bits_of_small_values():
    x = np.ldexp(np.random.default_rng(1).uniform(1, 2, 4096), -115).astype(np.float32)
    # (a bfloat16 has no bits below 2^-133)
    floor = lambda v: np.round(v * 2.0 ** 133) * 2.0 ** -133
    h, m, l = (floor(p) for p in _parts(x))
    assert np.any(h + m + l != x.astype(np.float64))


def test_what_is_left_out_of_a_product():
    rng = np.random.default_rng(2)
    x, y = (rng.uniform(1, 2, 1 << 20).astype(np.float32) for _ in range(2))
    exact = x.astype(np.float64) * y
    left = np.abs(_products(x, y) / exact - 1)
    assert left.max() < 2.0 ** -24 and np.sqrt(np.mean(left ** 2)) < 2.0 ** -27.4
    worst = np.array([1.0038986], np.float32)
    left = abs(float(_products(worst, worst)[0]) / float(worst[0]) ** 2 - 1)
    assert 2.0 ** -25 * 1.9 < left < 2.0 ** -24


@pytest.mark.parametrize("n", [88, 3600])
@pytest.mark.parametrize("missing", KEPT[1:])
def test_a_missing_product_shows_in_a_sum(n, missing):
    """2-norm over 256 sums of n products of one factor that is positive and one that is not, as in a weight gradient."""
    rng = np.random.default_rng(n)
    x = np.maximum(rng.normal(size=(256, n)), 0).astype(np.float32)
    y = rng.normal(size=(256, n)).astype(np.float32)
    exact = (x.astype(np.float64) * y).sum(1)
    err = lambda kept: np.linalg.norm(_products(x, y, kept).sum(1) - exact) / np.linalg.norm(exact)
    assert err(KEPT) < 2e-8
    assert err([k for k in KEPT if k != missing]) > 1.2e-6
