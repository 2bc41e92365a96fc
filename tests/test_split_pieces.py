"""What the batched FP32 form's contractions leave out: FP32 operands are split into three bf16
pieces, each the nearest to what the ones before leave, and of the nine piece products the three
smallest (mid lo, lo mid, lo lo) are not formed.  Over all 2^23 mantissas the pieces add up
exactly, and mid and lo stay below 2^-8 and 2^-17 of the value (a little above 2^-8 for mid), so
that what is left out of a product stays below 2^-24 of it, the rounding of an FP32 product.  A
leading piece rounded up or down at random would leave twice the remainder and not meet that."""
import numpy as np


def nearest(x):
    u = x.view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def at_random(x):  # the value's own lowest byte as the threshold
    u = x.view(np.uint32)
    return ((u + ((u & 0xff) << 8)) & 0xffff0000).view(np.float32)


def pieces(x, lead):
    hi = lead(x)
    mid = nearest(x - hi)
    lo = nearest(x - hi - mid)
    assert np.array_equal(hi.astype(np.float64) + mid + lo, x.astype(np.float64))
    return np.abs(mid) / x, np.abs(lo) / x


def test_products_left_out_are_below_fp32_rounding():
    x = (np.uint32(0x3f800000) + np.arange(1 << 23, dtype=np.uint32)).view(np.float32)
    mid, lo = pieces(x, nearest)
    # any operand's mid with any other's lo, both ways, and lo lo
    bound = 2.0 * mid.max() * lo.max() + lo.max() ** 2
    assert bound < 2.0 ** -24
    midr, lor = pieces(x, at_random)
    worst = np.argsort(-(midr * 2.0 ** 7 + lor * 2.0 ** 15))[:512]
    assert np.max(midr[worst][:, None] * lo.max()) + np.max(lor[worst]) * mid.max() > 2.0 ** -24
