"""LayerNorm at block sizes 64 and 128 in one pass over whole block rows: the narrowest and the widest rows, a ragged last strip,
several block rows per workgroup with a last one that does not exist, a second round of the persistent workgroups, both sides
of the bounds of layernorm_rows_fits."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from parity import assert_layernorm_param_grads_close
from test_gpu_parity import _check_eltwise, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,N,C", [(64, 64, 64), (64, 2048, 768), (64, 2048, 832), (64, 10240, 320), (64, 10176, 320), (64, 16448, 1024),
                                       (64, 8192, 1024), (64, 8128, 960), (64, 33024, 192), (64, 192, 1088), (128, 128, 128), (128, 2048, 384),
                                       (128, 20480, 256), (128, 20352, 256), (128, 33024, 512), (128, 16384, 512), (128, 16256, 512), (128, 256, 640)])
def test_layernorm_block_rows(block, N, C):
    eps = 1e-5
    say(f"layernorm block rows block={block} {N} x {C}")
    x, gamma, beta, gr = workloads.layernorm_case(9000 + C, N, C)
    (X, SX), (G, SG) = oracle.quantize_block(x, block), oracle.quantize_block(gr, block)
    Xd, SXd, Gd, SGd, gd, bd = map(dev, (X, SX, G, SG, gamma, beta))
    oY, oSY, omean, orstd, oy = oracle.layernorm_q(X, SX, gamma, beta, eps, block)
    atol = 1e-5 * np.abs(oracle.dequantize(X, SX, block)).max()
    Y, SY, mean, rstd = jf.jf_layernorm_q(Xd, SXd, gd, bd, eps, block)
    np.testing.assert_allclose(host(mean), omean, rtol=0, atol=atol)
    np.testing.assert_allclose(host(rstd), orstd, rtol=1e-5)
    _check_eltwise("forward", Y, SY, oY, oSY, oy, block)
    # the same rows from row partials: those of x + 0
    A, SA, row_mean, row_sumsq = jf.jf_add_q(Xd, SXd, torch.zeros_like(Xd), torch.zeros_like(SXd), block, want_partials=True)
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
    # in place: the same bits
    Xc, SXc = Xd.clone(), SXd.clone()
    jf.jf_layernorm_q(Xc, SXc, gd, bd, eps, block, out=(Xc, SXc, torch.empty_like(mean), torch.empty_like(rstd)))
    assert torch.equal(Xc, Y) and torch.equal(SXc, SY)
    Gc, SGc = Gd.clone(), SGd.clone()
    got = jf.jf_layernorm_q_bwd(Gc, SGc, Xd, SXd, gd, dev(omean), dev(orstd), block, out=(Gc, SGc, torch.empty_like(gd), torch.empty_like(gd)))
    assert torch.equal(got[0], dX) and torch.equal(got[1], SdX)
