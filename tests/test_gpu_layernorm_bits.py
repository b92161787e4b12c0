"""LayerNorm's codes and scales bit for bit: each of its kernels adds and multiplies in one order, and another order, though as accurate, moves
codes at rounding ties and with them block scales of the operators behind it (layernorm_chain).  A change of order has to be meant: it
changes the digests below, which were taken from kernels that tests/test_gpu_layernorm_*.py hold to the oracle."""
import hashlib

import numpy as np
import pytest

import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu

# block, N, C: forward, forward from an Add's row partials, backward.  One pass: column sums apart, twelve waves, sixteen waves, two teams,
# block rows of two and four teams; wider rows; the two-kernel scheme
DIGESTS = {
    (32, 512, 544): ("492684ee097d", "396244153b9a", "30ea82af9a39"),
    (32, 2080, 1280): ("b83bf3491a5a", "8ad959ed56d1", "8302523cdfc8"),
    (32, 2080, 2048): ("23233625f75d", "5d2c178186ef", "633deffca3da"),
    (32, 8256, 768): ("b2bedac22d30", "1d2455fe182c", "065d84b454d7"),
    (64, 10240, 704): ("848cb39e05cd", "d9356d4cc747", "94da121b6c4d"),
    (128, 20480, 384): ("44e7c3a13511", "e16251d48c78", "985e373533e6"),
    (32, 5120, 2304): ("8408202a884b", "810207c7facb", "8e11a73f9015"),
    (32, 256, 2304): ("69414a32a6a2", "2840da0c896a", "2689183823ac"),
    (64, 512, 1344): ("105d007b52d2", "a1a251a06299", "0a22c1387b8c"),
    (128, 384, 640): ("fd643132617f", "8c99b4ad1475", "d61aab28f846"),
}


def digests(block, N, C):
    g = workloads.rng(9950 + C)      # whole numbers and dyadic fractions: the same bits on every host
    codes = lambda: g.integers(-127, 128, (N, C), dtype=np.int8)
    fractions = lambda shape, low, high, unit: g.integers(low, high, shape).astype(np.float32) * np.float32(unit)
    scales = lambda: fractions((N // block, C // block), 100, 1000, 2.0 ** -16)
    X, SX, G, SG = map(dev, (codes(), scales(), codes(), scales()))
    gamma, beta, mean, rstd = map(dev, (fractions(C, 700, 1400, 2.0 ** -10), fractions(C, -100, 100, 2.0 ** -10), fractions(N, -200, 200, 2.0 ** -12),
                                        fractions(N, 500, 2000, 2.0 ** -10)))
    row_mean, row_sumsq = (dev(fractions((C // block, N), *r)) for r in ((-200, 200, 2.0 ** -12), (2000, 6000, block * 2.0 ** -14)))
    results = (jf.jf_layernorm_q(X, SX, gamma, beta, 1e-5, block), jf.jf_layernorm_q_partials(X, SX, row_mean, row_sumsq, gamma, beta, 1e-5, block),
               jf.jf_layernorm_q_bwd(G, SG, X, SX, gamma, mean, rstd, block))
    return tuple(hashlib.sha256(b"".join(host(t).tobytes() for t in r[:2])).hexdigest()[:12] for r in results)


@pytest.mark.parametrize("block,N,C", DIGESTS)
def test_codes_and_scales(block, N, C):
    say(f"bits block={block} {N} x {C}")
    assert digests(block, N, C) == DIGESTS[block, N, C]
