"""The arithmetic behind the products from bf16 pieces (csrc/kda_f32_tile.h), on the CPU: every fp32 significand splits exactly into three
bf16 pieces of the stated sizes, and the products of pieces that are left out are as small as stated."""
import numpy as np


def _bf16(x):
    """x rounded to the nearest bf16, ties to even, as an fp32 array (finite values)."""
    u = x.astype(np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


def _split(x):
    most = np.float32(float.fromhex("0x1.fep+127"))
    h = _bf16(np.clip(x, -most, most))
    m = _bf16(x - h)
    return h, m, _bf16(x - h - m)


def test_every_significand_is_the_exact_sum_of_its_pieces():
    x = np.arange(0x3F800000, 0x40000000, dtype=np.uint32).view(np.float32)       # [1, 2)
    h, m, l = (p.astype(np.float64) for p in _split(x))
    assert (h + m + l == x).all()
    assert (np.abs(m) <= 2.0 ** -8 * x).all() and (np.abs(l) <= 2.0 ** -17 * x).all()
    top = np.arange(0x7F000000, 0x7F800000, dtype=np.uint32).view(np.float32)     # the last binade, bf16's largest number within it
    h, m, l = (p.astype(np.float64) for p in _split(top))
    assert np.isfinite(h).all() and (h + m + l == top).all() and (np.abs(m) <= 2.0 ** 120).all()


def test_products_left_out_are_a_rounding_of_the_product():
    """m l' + l m' + l l' of two values: |m|, |m'| <= 2^-8 and |l|, |l'| <= 2^-17 of them make at most 2^-24 + 2^-34."""
    x = np.arange(0x3F800000, 0x40000000, dtype=np.uint32).view(np.float32)
    _, m, l = (p.astype(np.float64) for p in _split(x))
    rm, rl = m / x, l / x
    worst = np.argsort(-(np.abs(rm) + 512 * np.abs(rl)))[:2000]                   # the significands that can make it large
    worst = np.append(worst, int(0x00FF8 << 3))                                   # 1.00ff8 among them
    left = np.abs(np.outer(rm[worst], rl[worst]) + np.outer(rl[worst], rm[worst]) + np.outer(rl[worst], rl[worst]))
    assert 2.0 ** -24.1 < left.max() <= 2.0 ** -24 + 2.0 ** -34
