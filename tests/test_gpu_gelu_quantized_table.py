"""GELU forward looks quantized codes up: a block's largest result follows from its largest code, or from the two next to the lowest point of GELU.  It takes
FP32 tables where one block of the strip (of the workgroup, where its waves share blocks) has no ordinary scale or results next to none.  Blocks of every kind,
beside ordinary ones and beside one that forces the general way: codes and scales have to be the same both ways, and within the bound of the oracle."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu

# (scale, smallest code, largest code)
KINDS = {
    "both signs": (2.0 / 127, -127, 127),
    "positive decides just": (0.295 / 127, -127, 127),         # GELU(0.295) = 0.1817
    "small": (0.25 / 127, -127, 127),                          # the smallest code decides
    "negative alone, small": (0.69 / 127, -127, -1),
    "negative alone": (1.6 / 127, -127, -1),                   # the lowest point is in the middle
    "negative alone, large": (3.0 / 127, -127, -60),           # and here above the largest code
    "negative alone, lowest point at the end": (0.7517915 / 127, -127, -100),
    "negative alone, coarse": (2.5, -127, -1),
    "minus one": (1e-3, -1, 0),
    "small positive, large negative": (2.0 / 127, -127, 8),
    "far tail": (13.0 / 127, -127, -100),
    "beyond the tail": (0.16, -127, -80),                      # general: results from 1e-36 down to none
    "tiny": (1e-29, -127, 127),
    "subnormal": (1e-42, -127, 127),                           # general
    "zero scale": (0.0, -127, 127),
    "zero codes": (1.0, 0, 0),
    "one code": (0.01, 5, 5),
    "huge": (1e30, -127, 127),
    # results up to 3.05e38 and 3.3e38, of at most 3.4e38, that some lanes of the block have and others do not; and that all have
    "largest numbers": (2.4e36, -127, 127),
    "largest numbers, higher": (2.6e36, -127, 127),
    "largest numbers alone": (2.6e36, 118, 127),
}


def _block(g, kind, block):
    s, lo, hi = KINDS[kind]
    q = g.integers(lo, hi + 1, size=(block, block))
    q[0, 0], q[block - 1, block - 1] = lo, hi
    return q.astype(np.int8), np.float32(s)


def _tensor(g, block, rows, cols):
    names = list(KINDS)
    X, S, which = np.zeros((rows * block, cols * block), np.int8), np.zeros((rows, cols), np.float32), np.zeros((rows, cols), int)
    for i in range(rows):
        for j in range(cols):
            # ordinary blocks mostly, so that strips and workgroups of all quantized tables occur
            k = names[0] if g.random() < 0.5 and (i * cols + j) % 3 else names[(i * cols + j) // 3 % len(names)]
            which[i, j] = names.index(k)
            X[i * block:(i + 1) * block, j * block:(j + 1) * block], S[i, j] = _block(g, k, block)
    return X, S, which


# strips of four, two and one blocks, ragged; at block 32 and, but for the widest, at 64 on waves of 16 rows
@pytest.mark.parametrize("block,rows,cols", [(32, 16, 13), (32, 3, 1), (32, 120, 97), (64, 9, 5), (64, 40, 72), (128, 5, 3), (128, 14, 9)])
def test_blocks_of_every_kind(block, rows, cols):
    say(f"GELU tables block={block} {rows}x{cols} blocks")
    g = workloads.rng(9700 + block + rows)
    X, S, which = _tensor(g, block, rows, cols)
    Y, SY = jf.jf_gelu_q(dev(X), dev(S), block)
    y, sy = host(Y), host(SY)
    oY, oSY, of = oracle.gelu_q(X, S, block)
    ordinary = np.isin(which, [list(KINDS).index(k) for k in KINDS if k not in ("tiny", "subnormal", "huge", "far tail", "beyond the tail")])
    o = np.repeat(np.repeat(ordinary, block, 0), block, 1)
    np.testing.assert_allclose(sy[ordinary], oSY[ordinary], rtol=1e-5)
    d = np.abs(y.astype(int) - oY.astype(int))[o]
    assert d.max() <= 1 and np.count_nonzero(d) <= 1e-3 * d.size
    _same_the_general_way(X, S, block, y, sy)


def _large(g, block, rows, cols):
    """Such a tensor from copies of its first 37 rows of blocks."""
    X, S, _ = _tensor(g, block, 37, cols)
    return np.tile(X, (rows // 37 + 1, 1))[:rows * block], np.tile(S, (rows // 37 + 1, 1))[:rows]


# Waves of 32 rows, results written through, streamed and written back.  At block 32 each wave has its tables to itself and decides by itself.
LARGE = [(32, 480, 128), (32, 544, 128), (32, 352, 97), (64, 200, 64), (64, 272, 64), (64, 176, 49), (128, 120, 32), (128, 144, 32)]


@pytest.mark.parametrize("block,rows,cols", LARGE)
def test_large_tensors_of_every_kind(block, rows, cols):
    """The results of calls on parts that are small enough for waves of 16 rows (at block 128: for results that are written through)."""
    say(f"GELU tables, large, block={block} {rows}x{cols} blocks")
    X, S = _large(workloads.rng(9850 + block + rows), block, rows, cols)
    X, S = dev(X), dev(S)
    y, sy = jf.jf_gelu_q(X, S, block)
    part = 10_000_000 // (cols * block * block)
    for first in range(0, rows, part):
        r = slice(first, min(first + part, rows))
        py, psy = jf.jf_gelu_q(X[r.start * block:r.stop * block].contiguous(), S[r].contiguous(), block)
        np.testing.assert_array_equal(host(sy[r]), host(psy))
        np.testing.assert_array_equal(host(y[r.start * block:r.stop * block]), host(py))


def _same_the_general_way(X, S, block, y, sy):
    """The same blocks beside one of a negative scale in each strip, which forces it the general way, have the results y and sy."""
    X2, S2 = X.copy(), S.copy()
    first = np.zeros(S.shape, bool)
    for c in range(0, S.shape[1], 128 // block):
        first[:, c] = True
        X2[:, c * block:(c + 1) * block] = -100
        S2[:, c] = -0.02
    Y2, SY2 = jf.jf_gelu_q(dev(X2), dev(S2), block)
    keep = ~first
    k = np.repeat(np.repeat(keep, block, 0), block, 1)
    np.testing.assert_array_equal(host(SY2)[keep], sy[keep])
    np.testing.assert_array_equal(host(Y2)[k], y[k])


@pytest.mark.parametrize("block,rows,cols", [(32, 96, 128), (64, 64, 34)])
def test_blocks_without_a_large_code(block, rows, cols):
    """The codes about the lowest point of GELU at -0.75 decide: of every scale and range of codes, with gaps, some also in the far tail."""
    say(f"GELU negative blocks block={block} {rows}x{cols} blocks")
    g = workloads.rng(9800 + block)
    S = np.exp(g.uniform(np.log(1e-4), np.log(0.2), size=(rows, cols))).astype(np.float32)
    lo = g.integers(-127, 1, size=S.shape)
    hi = np.minimum(lo + g.integers(0, 128, size=S.shape), (0.28 / S).astype(int))
    up = lambda a: np.repeat(np.repeat(a, block, 0), block, 1)
    X = g.integers(up(lo), up(hi) + 1)
    X = np.where((X % 16 < 12) | up(g.random(S.shape) < 0.5), X, up(lo)).astype(np.int8)
    y, sy = (host(t) for t in jf.jf_gelu_q(dev(X), dev(S), block))
    oY, oSY, _ = oracle.gelu_q(X, S, block)
    # The oracle's 1 + erf(x / sqrt 2) is off by up to 2^-53 and an input reaches 25: 25 * 2^-54 / 127 = 1.1e-17 of a scale, 1e-6 of one of 1e-11.
    near = oSY > 1e-11
    np.testing.assert_allclose(sy[near], oSY[near], rtol=1e-5)
    d = np.abs(y.astype(int) - oY.astype(int))[up(near)]
    assert d.max() <= 1 and np.count_nonzero(d) <= 1e-3 * d.size
    _same_the_general_way(X, S, block, y, sy)


@pytest.mark.parametrize("block,rows,cols", [(32, 8, 8), (64, 8, 8), (128, 8, 8), (32, 480, 128), (32, 352, 97)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, -0.5])
def test_scales_that_are_none(block, rows, cols, bad):
    """A block with such a scale leaves the others of its strip and workgroup what they are without it."""
    say(f"GELU tables block={block} {rows}x{cols} blocks, scale {bad}")
    g = workloads.rng(9750 + block)
    X, S = _large(g, block, rows, cols)
    y, sy = (host(t) for t in jf.jf_gelu_q(dev(X), dev(S), block))
    S2 = S.copy()
    S2[3, 2] = bad
    y2, sy2 = (host(t) for t in jf.jf_gelu_q(dev(X), dev(S2), block))
    keep = np.ones(S.shape, bool)
    keep[3, 2] = False
    k = np.repeat(np.repeat(keep, block, 0), block, 1)
    np.testing.assert_array_equal(sy2[keep], sy[keep])
    np.testing.assert_array_equal(y2[k], y[k])


@pytest.mark.parametrize("block", [32, 64, 128])
def test_scales_of_blocks_without_results(block):
    """Codes or scales of 0, or inputs so far below 0 that GELU is 0: the scale is 0 and not -0, beside ordinary blocks and alone."""
    say(f"GELU blocks without results, block={block}")
    g = workloads.rng(9950 + block)
    S = np.tile(np.array([0.02, 0.0, 1.0, 2.0], np.float32), (6, 2))
    X = g.integers(-127, 128, size=(6 * block, 8 * block))
    X[:, 2 * block:3 * block] = X[:, 6 * block:7 * block] = 0
    X[:, 3 * block:4 * block] = X[:, 7 * block:] = -100
    X[2 * block:], S[2:] = -100, 2.0
    sy = host(jf.jf_gelu_q(dev(X.astype(np.int8)), dev(S), block)[1])
    ordinary = np.zeros(S.shape, bool)
    ordinary[:2, ::4] = True
    assert (sy[ordinary] > 0).all() and not sy[~ordinary].any() and not np.signbit(sy).any()
