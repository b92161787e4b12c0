"""A scale that is infinite or not a number makes the results unspecified that are formed from its block, and no others: what does not depend on
the block is bit for bit as without it, where the lanes of a wave reduce the values of several blocks together and where workgroups share rows."""
import pytest
import torch

import paper_2403_12422_amd as jf
from test_gpu_parity import say

pytestmark = pytest.mark.gpu
BAD = [float("inf"), float("nan")]


def _with(s, at, value):
    s = s.clone()
    s[at] = value
    return s


# a block amid the tiles and, at these sizes, in a ragged last one of every shape
@pytest.mark.parametrize("value", BAD)
@pytest.mark.parametrize("block,shape", [(32, s) for s in (1, 4, 6, 7, 8, 10)] + [(64, s) for s in (1, 4, 11)] + [(128, s) for s in (1, 6, 11)])
def test_product(block, shape, value):
    say(f"not finite: product block {block} shape {shape} {value}")
    g = torch.Generator(device="cuda").manual_seed(5100)
    N, C, D = 11 * block, 5 * block, 13 * block
    x, w = (jf.jf_quantize_block(torch.randn((r, C), generator=g, device="cuda"), block) for r in (N, D))
    jf.jf_debug_set_gemm_shape(shape)
    try:
        want = jf.jf_linear_fwd(*x, *w, block)
        for row in (2, 10):
            got = jf.jf_linear_fwd(x[0], _with(x[1], (row, 3), value), *w, block)
            rows, grid = torch.ones(N, dtype=torch.bool, device="cuda"), torch.ones(N // block, dtype=torch.bool, device="cuda")
            rows[row * block:(row + 1) * block] = False
            grid[row] = False
            assert torch.equal(got[0][rows], want[0][rows]) and torch.equal(got[1][grid], want[1][grid])
    finally:
        jf.jf_debug_set_gemm_shape(0)


# row groups shared by four workgroups, by two (column sums apart, and as partial rows), and not shared
@pytest.mark.parametrize("value", BAD)
@pytest.mark.parametrize("N,C", [(96, 160), (1056, 800), (2048, 768), (3840, 512), (4096, 2048), (8192, 640)])
def test_layernorm(N, C, value):
    say(f"not finite: layernorm {N} x {C} {value}")
    B = 32
    g = torch.Generator(device="cuda").manual_seed(5200 + N)
    x, dy = (jf.jf_quantize_block(torch.randn((N, C), generator=g, device="cuda"), B) for _ in range(2))
    gamma, beta = (1.0 + 0.1 * torch.randn((C,), generator=g, device="cuda") for _ in range(2))
    want = jf.jf_layernorm_q(*x, gamma, beta, 1e-5, B)
    want_bwd = jf.jf_layernorm_q_bwd(*dy, *x, gamma, want[2], want[3], B)
    for row, col in ((1, 1), (N // B - 1, C // B - 1)):
        rows, grid = torch.ones(N, dtype=torch.bool, device="cuda"), torch.ones(N // B, dtype=torch.bool, device="cuda")
        rows[row * B:(row + 1) * B] = False
        grid[row] = False
        cols = torch.ones(C, dtype=torch.bool, device="cuda")
        cols[col * B:(col + 1) * B] = False
        got = jf.jf_layernorm_q(x[0], _with(x[1], (row, col), value), gamma, beta, 1e-5, B)
        for a, b, keep in zip(got, want, (rows, grid, rows, rows)):
            assert torch.equal(a[keep], b[keep])
        for bad in ((dy[0], _with(dy[1], (row, col), value), *x), (*dy, x[0], _with(x[1], (row, col), value))):
            got = jf.jf_layernorm_q_bwd(*bad, gamma, want[2], want[3], B)
            for a, b, keep in zip(got, want_bwd, (rows, grid, cols, cols)):
                assert torch.equal(a[keep], b[keep])
