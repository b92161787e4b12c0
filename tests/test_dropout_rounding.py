"""Dropout rounds with one FP32 FMA: the code times 127 / max|code|, that factor moved to one side by 2^-20 of itself.  The rule against the exact
quotient of the FP32 numbers: for every code and every maximum at a sample of the scales, the binades at the rule's ends among them, and for the codes
at and beside half an even maximum, the only tie there is, at every significand of the scale."""
import numpy as np

F32 = np.float32


def _codes(k, m, c=None):
    """k (n,) float32, m the largest |code|: codes c, or all, by the rule and by round-half-even of the exact quotient."""
    c = np.arange(-m, m + 1) if c is None else c
    amax = (F32(m) * k).astype(F32)
    s = amax / F32(127)
    over = np.sign(s.astype(np.float64) * 127 - amax)                                # exact: 24 bits times 7
    for reciprocal in (np.nextafter(F32(1) / F32(m), F32(0)), F32(1) / F32(m), np.nextafter(F32(1) / F32(m), F32(2))):   # within an ulp of it
        f = F32(127) * reciprocal * np.where(over > 0, F32(1 - 2.0 ** -20), F32(1 + 2.0 ** -20))
        rule = np.rint(c[None, :] * f[:, None].astype(np.float64))                   # 8 by 24 bits are exact in a double: one rounding, as the FMA's
        y = (c[None, :].astype(F32) * k[:, None]).astype(np.float64)
        q = y / s[:, None].astype(np.float64)                                        # a tie or at least 2^-26 away from one
        np.testing.assert_array_equal(rule, np.rint(q), err_msg=f"m = {m}")


def test_every_code_and_maximum():
    g = np.random.default_rng(5)
    for m in range(1, 129):
        k = np.exp2(g.integers(-100, 100, 300)) * (1 + g.random(300))
        k = np.concatenate([k.astype(F32), (1 + np.arange(32) / 32).astype(F32), 127 * np.exp2(np.arange(-60.0, 60, 7)).astype(F32), [F32(2.0 ** -100), F32(2.0 ** 100)]])
        _codes(k.astype(F32), m)


def test_significands_at_every_even_maximum():
    for m in range(2, 129, 2):
        _codes(np.arange((1 << 23) + m, 1 << 24, 4099).astype(F32), m)


def test_ties_at_every_significand():
    for m in (2, 64, 126):
        for first in range(1 << 23, 1 << 24, 1 << 20):
            _codes(np.arange(first, first + (1 << 20)).astype(F32), m, np.arange(m // 2 - 1, m // 2 + 2))
