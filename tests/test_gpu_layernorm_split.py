"""LayerNorm of few row groups at block size 32, each shared by several workgroups: the codes, scales and statistics of the kernels that keep
a row group to one workgroup, bit for bit, and the column sums of the oracle.  With an output over an input the calls take the latter."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from parity import assert_layernorm_param_grads_close
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu
EPS, BLOCK = 1e-5, 32


# one block, one group; a ragged last strip; groups that are no multiple of eight; four parts, two, and where they end, forward (1024 and 4096
# rows) and backward (by the columns: 2048 x 768 and 1792 x 512); column sums as partial rows from 2592 x 1536 and behind 3072 x 2048 on
@pytest.mark.parametrize("N,C", [(32, 32), (32, 2048), (96, 160), (1024, 800), (1056, 800), (1056, 160), (1792, 512), (1824, 96), (2048, 768), (2560, 1536),
                                 (2592, 1536), (3072, 2048), (3104, 1952), (3840, 512), (3872, 512), (4064, 2048), (4096, 352), (4128, 352)])
def test_parts_of_a_row_group(N, C):
    say(f"layernorm split {N} x {C}")
    g = workloads.rng(9300 + N + C)
    (X, SX), (G, SG) = (oracle.quantize_block(workloads.gaussian(g, N, C, std), BLOCK) for std in (1.0, 1e-3))
    gamma, beta = ((m + 0.1 * g.standard_normal(C, dtype=np.float32)).astype(np.float32) for m in (1.0, 0.0))
    Xd, SXd, Gd, SGd, gd, bd = map(dev, (X, SX, G, SG, gamma, beta))
    zero = torch.zeros_like(Xd), torch.zeros_like(SXd)
    partials = jf.jf_add_q(Xd, SXd, *zero, BLOCK, want_partials=True)[2:]
    row = lambda: torch.empty((N,), dtype=torch.float32, device="cuda")

    def over(x, sx):   # outputs over these inputs
        return x.clone(), sx.clone()

    for forward in (lambda x, sx, out=None: jf.jf_layernorm_q(x, sx, gd, bd, EPS, BLOCK, out=out),
                    lambda x, sx, out=None: jf.jf_layernorm_q_partials(x, sx, *partials, gd, bd, EPS, BLOCK, out=out)):
        got = forward(Xd, SXd)
        x, sx = over(Xd, SXd)
        for a, b in zip(got, forward(x, sx, out=(x, sx, row(), row()))):
            assert torch.equal(a, b)
    Y, SY, mean, rstd = jf.jf_layernorm_q(Xd, SXd, gd, bd, EPS, BLOCK)
    got = jf.jf_layernorm_q_bwd(Gd, SGd, Xd, SXd, gd, mean, rstd, BLOCK)
    x, sx = over(Xd, SXd)
    sums = (torch.empty((C,), dtype=torch.float32, device="cuda") for _ in range(2))
    want = jf.jf_layernorm_q_bwd(Gd, SGd, x, sx, gd, mean, rstd, BLOCK, out=(x, sx, *sums))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    o = oracle.layernorm_q_bwd(G, SG, X, SX, gamma, host(mean), host(rstd), BLOCK)
    xh = (oracle.dequantize(X, SX, BLOCK) - host(mean)[:, None].astype(np.float64)) * host(rstd)[:, None].astype(np.float64)
    assert_layernorm_param_grads_close(host(got[2]), host(got[3]), o[2], o[3], oracle.dequantize(G, SG, BLOCK), xh, "layernorm bwd")
