"""Dropout on blocks of every largest code, with half of it (63.5 scales) among the elements, and on scales at the ends of what its one-FMA rounding
takes and beyond them: zero, subnormal, the largest, negative; codes and scales are those of the operator
in FP32 with Eq. 1's quotient rounded exactly."""
import numpy as np
import pytest

import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


def _fp32(X, S, keep, p, block):
    """The operator in FP32, Eq. 1's quotient rounded exactly: y = fl(code k), k = fl(scale fl(1 / (1 - p)))."""
    up = lambda a: np.repeat(np.repeat(a, block, 0), block, 1)
    k = (S * np.float32(1.0 / (1.0 - float(np.float32(p))))).astype(np.float32)
    y = np.where(keep, X, 0).astype(np.float32) * up(k)
    amax = np.abs(y).reshape(S.shape[0], block, S.shape[1], block).max(axis=(1, 3))
    s = (amax / np.float32(127)).astype(np.float32)
    d = up(s).astype(np.float64)
    return np.rint(np.divide(y.astype(np.float64), d, out=np.zeros_like(d), where=d > 0)).astype(np.int8), s


def _check(X, S, p, block, g):
    keep = g.random(X.shape) >= p
    Y, SY = jf.jf_dropout_q(dev(X), dev(S), dev(np.packbits(keep, axis=1, bitorder="little")), p, block)
    y, s = _fp32(X, S, keep, p, block)
    np.testing.assert_array_equal(host(SY), s)
    np.testing.assert_array_equal(host(Y), y)


def _blocks(g, block, largest):
    rows, cols = len(largest) * block, 3 * block
    X = np.zeros((rows, cols), np.int8)
    for i, m in enumerate(largest):
        b = g.integers(-m, m + 1, size=(block, cols))
        b = np.where(g.random(b.shape) < 0.1, g.choice([-m, m], b.shape), b)
        b = np.where(g.random(b.shape) < 0.2, g.choice([-(m // 2), m // 2, (m + 1) // 2], b.shape), b)
        X[i * block:(i + 1) * block] = b
    return X


@pytest.mark.parametrize("block", [32, 64, 128])
@pytest.mark.parametrize("p", [0.0, 0.1, 0.9995])
def test_every_largest_code(block, p):
    say(f"dropout block={block} p={p}: every largest code")
    g = workloads.rng(9900 + block)
    largest = list(range(0, 128)) if block == 32 else list(range(0, 128, 3)) + [126, 127]
    X = _blocks(g, block, largest)
    S = np.exp2(g.uniform(-20, 20, (len(largest), 3))).astype(np.float32)
    _check(X, S, p, block, g)


@pytest.mark.parametrize("block", [32, 64, 128])
def test_scales_at_the_ends(block):
    say(f"dropout block={block}: scales at the ends")
    g = workloads.rng(9950 + block)
    ends = [0.0, 1e-45, 1e-42, 2.0 ** -126, 2.0 ** -101, 2.0 ** -100, 2.0 ** -99, 2.0 ** 99, 2.0 ** 100, 2.0 ** 101, 2.0 ** 118, -1.0, -2.0 ** -120, 1.0]
    X = _blocks(g, block, [127, 126, 64, 3] * len(ends))
    S = np.repeat(np.array(ends, np.float32), 12).reshape(-1, 3)
    S[:, 1] = 1.5                                            # beside an ordinary block in the same wave
    _check(X, S, 0.25, block, g)
