"""The quantizer on FP16 where its quotients are ties: a block for every significand of the maximum, half of the maximum (63.5 scales) among its
elements, all ties that a scale of few bits has, and the neighbours of both; codes and scales are the oracle's."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", [0, 1, 15, 30])
@pytest.mark.parametrize("block", [32, 64, 128])
def test_every_significand(block, exponent):
    say(f"quantize FP16 block={block} exponent {exponent}")
    g = workloads.rng(9800 + block + exponent)
    step = 1024 // (32 * 128 // block)                       # every significand at block 32, at larger blocks a part of them
    sig = np.union1d(np.arange(0 if exponent else 1, 1024, step), 127 * np.arange(9, 17)[127 * np.arange(9, 17) < 2048] - 1024)
    bits = (exponent * 1024 + sig).astype(np.uint16)
    bits = np.resize(bits, -(-len(bits) // 3) * 3)
    amax = bits.view(np.float16)
    x = np.empty((block * (len(bits) // 3), 3 * block), np.float16)
    for n, a in enumerate(amax):
        # half steps of the scale, their FP16 neighbours, and any smaller number
        k = g.integers(-254, 255, size=(block, block)) * (float(a) / 254)
        t = k.astype(np.float16)
        t = (t.view(np.uint16) + g.integers(-1, 2, size=t.shape) * (t != 0)).astype(np.uint16).view(np.float16)
        other = (g.random((block, block)) * 2 - 1) * float(a)
        t = np.where(g.random(t.shape) < 0.5, t, other.astype(np.float16))
        t = np.clip(t, -a, a)
        t[3, 5], t[block - 1, 0], t[0, block - 1] = a, a / np.float16(2), -a / np.float16(2)
        i, j = divmod(n, 3)
        x[i * block:(i + 1) * block, j * block:(j + 1) * block] = t
    oq, os_ = oracle.quantize_block(x.astype(np.float32), block)
    q, s = jf.jf_quantize_block(dev(x), block)
    np.testing.assert_array_equal(host(s), os_)
    np.testing.assert_array_equal(host(q), oq)
    q, s, qt, st = jf.jf_quantize_block(dev(x), block, transposed_copy=True)
    np.testing.assert_array_equal(host(q), oq)
    np.testing.assert_array_equal(host(qt), oq.T)
    np.testing.assert_array_equal(host(st), os_.T)
