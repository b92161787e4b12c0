"""LayerNorm's codes and scales bit for bit: each of its kernels adds and multiplies in one order, and another order, though as accurate, moves
codes at rounding ties and with them block scales of the operators behind it (layernorm_chain).  A change of order has to be meant: it
changes the digests below, which were taken from kernels that tests/test_gpu_layernorm_*.py hold to the oracle."""
import hashlib

import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu

# block, N, C: forward, forward from an Add's row partials, backward.  One pass: column sums apart, twelve waves, sixteen waves, two teams,
# block rows of two and four teams; wider rows; the two-kernel scheme
DIGESTS = {
    (32, 512, 544): ("c2fcdfcf3714", "1d834f156566", "1e56b8cf1f42"),
    (32, 2080, 1280): ("1958cfd68f18", "0cd1229e26ee", "4834888946ac"),
    (32, 2080, 2048): ("177c063967cb", "05199eb0f385", "daa2f5022244"),
    (32, 8256, 768): ("a1f6c749e345", "fd8d97b86dd6", "8e24002f3c53"),
    (64, 10240, 704): ("85322718c4cd", "e0a1adca7747", "503e83d0b4ca"),
    (128, 20480, 384): ("b3d85cced972", "b00c9a3be215", "1ceed59ff66c"),
    (32, 5120, 2304): ("de0aebb446ba", "e2cc92db6952", "5d06ff33587d"),
    (32, 256, 2304): ("e426efa98c34", "b363ce690b71", "ff601c371dfa"),
    (64, 512, 1344): ("3def0e919c73", "750877147823", "71bff7c28f70"),
    (128, 384, 640): ("4e5f01024eb6", "cf524e6d60b5", "36dd74125c14"),
}


def digests(block, N, C):
    x, gamma, beta, gr = workloads.layernorm_case(9950 + C, N, C)
    (X, SX), (G, SG) = oracle.quantize_block(x, block), oracle.quantize_block(gr, block)
    mean, rstd = oracle.layernorm_q(X, SX, gamma, beta, 1e-5, block)[2:4]
    row_mean, row_sumsq = oracle.add_q(X, SX, np.zeros_like(X), np.zeros_like(SX), block)[2:4]
    X, SX, G, SG, gamma, beta, mean, rstd = map(dev, (X, SX, G, SG, gamma, beta, mean, rstd))
    results = (jf.jf_layernorm_q(X, SX, gamma, beta, 1e-5, block),
               jf.jf_layernorm_q_partials(X, SX, dev(row_mean.T), dev(row_sumsq.T), gamma, beta, 1e-5, block),
               jf.jf_layernorm_q_bwd(G, SG, X, SX, gamma, mean, rstd, block))
    return tuple(hashlib.sha256(b"".join(host(t).tobytes() for t in r[:2])).hexdigest()[:12] for r in results)


@pytest.mark.parametrize("block,N,C", DIGESTS)
def test_codes_and_scales(block, N, C):
    say(f"bits block={block} {N} x {C}")
    assert digests(block, N, C) == DIGESTS[block, N, C]
