"""LayerNorm at block size 32 in one pass over rows of more than 2048 columns: one strip more than full steps, waves without a last
step, the narrowest and the widest rows, a second and a third round of the persistent workgroups with an incomplete last one, both sides
of the bounds of layernorm_wide_fits."""
import pytest
import torch

import paper_2403_12422_amd as jf
import test_gpu_layernorm_block_rows as block_rows
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C", [(5120, 2080), (5088, 2080), (8192, 2176), (8224, 2080), (5152, 3104), (5120, 4128), (10240, 2080), (11264, 2080), (13120, 2112),
                                 (16672, 2080), (5120, 7168), (5120, 7200)])
def test_layernorm_wide_rows(N, C):
    block_rows.test_layernorm_block_rows(32, N, C)


@pytest.mark.parametrize("N,C", [(5120, 11264), (5120, 8192)])
def test_widest_rows_backward(N, C):
    """Against double precision; in place over either operand."""
    say(f"layernorm backward wide rows {N} x {C}")
    g = torch.Generator(device="cuda")
    g.manual_seed(N + C)
    X = torch.randint(-127, 128, (N, C), dtype=torch.int8, device="cuda", generator=g)
    G = torch.randint(-127, 128, (N, C), dtype=torch.int8, device="cuda", generator=g)
    SX, SG = (torch.rand((N // 32, C // 32), device="cuda", generator=g) * 0.01 + 1e-3 for _ in range(2))
    mean, rstd = torch.randn((N,), device="cuda", generator=g) * 0.1, torch.rand((N,), device="cuda", generator=g) + 0.5
    gamma = torch.randn((C,), device="cuda", generator=g)
    dX, SdX, dgamma, dbeta = jf.jf_layernorm_q_bwd(G, SG, X, SX, gamma, mean, rstd, 32)
    q1 = q2 = 0.0
    parts = []
    for c in range(0, C, 1024):   # double precision, a range of columns at a time
        cs, bs = slice(c, c + 1024), slice(c // 32, c // 32 + 32)
        up = lambda t, s: t[:, cs].double() * s[:, bs].double().repeat_interleave(32, 0).repeat_interleave(32, 1)
        gv, xh = up(G, SG), (up(X, SX) - mean.double()[:, None]) * rstd.double()[:, None]
        gh = gv * gamma[cs].double()
        q1, q2 = q1 + gh.sum(1), q2 + (gh * xh).sum(1)
        bound = 4 * N * 2.0 ** -24   # FP32 sums of N terms with a few roundings each
        assert ((dgamma[cs] - (gv * xh).sum(0)).abs() <= bound * (gv * xh).abs().sum(0)).all()
        assert ((dbeta[cs] - gv.sum(0)).abs() <= bound * gv.abs().sum(0)).all()
        parts.append((cs, bs, gh, xh))
    for cs, bs, gh, xh in parts:
        want = rstd.double()[:, None] * (gh - (q1 / C)[:, None] - xh * (q2 / C)[:, None])
        scale = want.abs().reshape(N // 32, 32, 32, 32).amax(dim=(1, 3)) / 127.0
        assert ((SdX[:, bs] - scale).abs() <= 2e-5 * scale).all()
        got = dX[:, cs].double() * SdX[:, bs].double().repeat_interleave(32, 0).repeat_interleave(32, 1)
        wide = SdX[:, bs].double().repeat_interleave(32, 0).repeat_interleave(32, 1)
        assert ((got - want).abs() <= (0.5 + 3e-3) * wide).all()   # half a step, and FP32 evaluation (2e-5 of 127 steps)
    # in place: the same bits
    for out in ((G.clone(), SG.clone()), (X.clone(), SX.clone())):
        g_in = out if torch.equal(out[0], G) else (G, SG)
        x_in = out if torch.equal(out[0], X) else (X, SX)
        got = jf.jf_layernorm_q_bwd(*g_in, *x_in, gamma, mean, rstd, 32, out=(*out, torch.empty_like(gamma), torch.empty_like(gamma)))
        for a, b in zip(got, (dX, SdX, dgamma, dbeta)):
            assert torch.equal(a, b)
