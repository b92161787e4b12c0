"""LayerNorm backward where the column sums come from workgroups of their own: in front of the two-kernel scheme's tiles, and
behind the row workgroups of short tensors at block size 32 (up to 2048 rows, up to 12 row groups per wave)."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from parity import assert_layernorm_param_grads_close
from test_gpu_parity import _check_eltwise, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,N,C", [(32, 32, 32), (32, 384, 128), (32, 416, 128), (32, 768, 160), (32, 800, 160), (32, 2048, 704),
                                       (32, 2080, 704), (32, 1024, 2048), (32, 96, 2080), (64, 64, 64), (64, 1088, 320), (128, 384, 1152)])
def test_column_sums(block, N, C):
    say(f"layernorm backward block={block} {N} x {C}")
    g = workloads.rng(6100 + N + C)
    X, SX = oracle.quantize_block(workloads.gaussian(g, N, C, 1.0), block)
    G, SG = oracle.quantize_block(workloads.gaussian(g, N, C, 1e-3), block)
    gamma = (1.0 + 0.1 * g.standard_normal(C, dtype=np.float32)).astype(np.float32)
    mean, rstd = oracle.layernorm_q(X, SX, gamma, np.zeros(C, np.float32), 1e-5, block)[2:4]
    o = oracle.layernorm_q_bwd(G, SG, X, SX, gamma, mean, rstd, block)
    args = tuple(map(dev, (G, SG, X, SX, gamma, mean, rstd)))
    got = jf.jf_layernorm_q_bwd(*args, block)
    _check_eltwise("layernorm bwd", got[0], got[1], o[0], o[1], o[4], block)
    xh = (oracle.dequantize(X, SX, block) - mean[:, None].astype(np.float64)) * rstd[:, None].astype(np.float64)
    assert_layernorm_param_grads_close(host(got[2]), host(got[3]), o[2], o[3], oracle.dequantize(G, SG, block), xh, "layernorm bwd")
    for a, b in zip(got, jf.jf_layernorm_q_bwd(*args, block)):   # fixed summation orders
        np.testing.assert_array_equal(host(a), host(b))
