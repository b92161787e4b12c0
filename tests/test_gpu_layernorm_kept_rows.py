"""LayerNorm backward at block size 32 on workgroups of at most 12 waves, which keep ghat of some rows in registers: one team of
ten and of twelve waves with and without a second row group, two teams of six with a last one that has no rows, and all four
rows kept where the column sums are taken apart."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from parity import assert_layernorm_param_grads_close
from test_gpu_parity import _check_eltwise, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C", [(2080, 1280), (8256, 1536), (16416, 768), (2080, 96), (2048, 1248)])
def test_layernorm_backward(N, C):
    block = 32
    say(f"layernorm backward {N} x {C}")
    x, gamma, beta, gr = workloads.layernorm_case(8900 + C, N, C)
    (X, SX), (G, SG) = oracle.quantize_block(x, block), oracle.quantize_block(gr, block)
    mean, rstd = oracle.layernorm_q(X, SX, gamma, beta, 1e-5, block)[2:4]
    dX, SdX, dgamma, dbeta = jf.jf_layernorm_q_bwd(*map(dev, (G, SG, X, SX, gamma, mean, rstd)), block)
    o = oracle.layernorm_q_bwd(G, SG, X, SX, gamma, mean, rstd, block)
    _check_eltwise("backward", dX, SdX, o[0], o[1], o[4], block)
    xh = (oracle.dequantize(X, SX, block) - mean[:, None].astype(np.float64)) * rstd[:, None].astype(np.float64)
    assert_layernorm_param_grads_close(host(dgamma), host(dbeta), o[2], o[3], oracle.dequantize(G, SG, block), xh, "backward")
