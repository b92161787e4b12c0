"""The FP16 quantizer rounds with one FP32 multiplication by a reciprocal that is moved to the right side of 127 / max|x|.  That rule against
the exact quotient, for every FP16 significand of the block's maximum and every FP16 value below it that does not round to 0 at once."""
import numpy as np


def _ulp(f, steps):
    return (f.view(np.int32) + steps).view(np.float32)


def _pairs_agree(amax, x):
    """amax (n,), x (n, m) in float16: the rule's code and round-half-even of the exact x / s."""
    a = amax.astype(np.float32)
    s = a / np.float32(127)
    over = np.sign(s.astype(np.float64) * 127 - a)                                   # exact: 24 bits times 7
    near = (1.0 / s.astype(np.float64)).astype(np.float32)
    inv = _ulp(near, np.where(over > 0, -1, np.where(over < 0, 1, 0)).astype(np.int32))
    one_fma = ~((over == 0) & ((s.view(np.int32) & 0x7fffff) != 0))                  # the others take the exact rounding
    exact = np.rint(x.astype(np.float64) / s.astype(np.float64)[:, None])            # a quotient is a tie or at least 2^-26 away from one
    fma = np.rint(x.astype(np.float64) * inv.astype(np.float64)[:, None])            # 11 by 24 bits are exact in a double: one rounding
    assert (fma == exact)[one_fma].all()
    return one_fma


def test_every_significand():
    bits = np.arange(0x7800, 0x7c00, dtype=np.uint16)                                # the largest binade
    amax = bits.view(np.float16)
    taken = 0
    for down in range(10):                                                           # 2^-9 of the maximum rounds to 0
        x = (bits - np.uint16(down * 0x400)).view(np.float16)
        x = np.minimum(x[None, :], amax[:, None])
        taken += _pairs_agree(amax, np.concatenate([x, -x], axis=1)).sum()
    assert taken == 10 * (1024 - 7)                                                  # all but 9, 10 .. 15 times 127


def test_subnormal_maxima():
    bits = np.arange(1, 0x800, dtype=np.uint16)                                      # subnormals and the first binade
    amax = bits.view(np.float16)
    x = np.minimum(amax[None, :], amax[:, None])
    _pairs_agree(amax, np.concatenate([x, -x], axis=1))
