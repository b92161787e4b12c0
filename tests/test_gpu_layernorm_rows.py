"""LayerNorm at block size 32 in one pass over whole rows: the edges of its range -- one block, a ragged last strip, several
teams of waves per workgroup with a last team that has no rows, a second round of the persistent workgroups, the widest
row that the compute unit's LDS holds and the first that it does not (run with -m gpu)."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from parity import assert_layernorm_param_grads_close
from test_gpu_parity import _check_eltwise, dev, host, say

import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C", [(32, 32), (96, 128), (96, 1920), (8256, 2048), (96, 2080), (66592, 160), (9248, 640), (24672, 384),
                                 (1056, 800)])
def test_layernorm_rows(N, C):
    block, eps = 32, 1e-5
    say(f"layernorm rows {N}x{C}")
    x, gamma, beta, gr = workloads.layernorm_case(8800 + C, N, C)
    (X, SX), (G, SG) = oracle.quantize_block(x, block), oracle.quantize_block(gr, block)
    Xd, SXd, Gd, SGd, gd, bd = map(dev, (X, SX, G, SG, gamma, beta))
    oY, oSY, omean, orstd, oy = oracle.layernorm_q(X, SX, gamma, beta, eps, block)
    atol = 1e-5 * np.abs(oracle.dequantize(X, SX, block)).max()
    Y, SY, mean, rstd = jf.jf_layernorm_q(Xd, SXd, gd, bd, eps, block)
    np.testing.assert_allclose(host(mean), omean, rtol=0, atol=atol)
    np.testing.assert_allclose(host(rstd), orstd, rtol=1e-5)
    _check_eltwise("forward", Y, SY, oY, oSY, oy, block)
    # the same rows from row partials: those of x + 0
    zero = torch.zeros_like(Xd), torch.zeros_like(SXd)
    A, SA, row_mean, row_sumsq = jf.jf_add_q(Xd, SXd, *zero, block, want_partials=True)
    assert torch.equal(A, Xd)
    Z, SZ, mean, rstd = jf.jf_layernorm_q_partials(A, SA, row_mean, row_sumsq, gd, bd, eps, block)
    np.testing.assert_allclose(host(mean), omean, rtol=0, atol=atol)
    np.testing.assert_allclose(host(rstd), orstd, rtol=1e-5)
    _check_eltwise("from partials", Z, SZ, oY, oSY, oy, block)
    dX, SdX, dgamma, dbeta = jf.jf_layernorm_q_bwd(Gd, SGd, Xd, SXd, gd, dev(omean), dev(orstd), block)
    odX, oSdX, odg, odb, odx = oracle.layernorm_q_bwd(G, SG, X, SX, gamma, omean, orstd, block)
    _check_eltwise("backward", dX, SdX, odX, oSdX, odx, block)
    xh = (oracle.dequantize(X, SX, block) - omean[:, None].astype(np.float64)) * orstd[:, None].astype(np.float64)
    assert_layernorm_param_grads_close(host(dgamma), host(dbeta), odg, odb, oracle.dequantize(G, SG, block), xh, "backward")
