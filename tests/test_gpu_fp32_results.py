"""FP32 results without codes leave a tile by way of LDS, in whole lines (256x256 tiles: from each lane, as beside codes); beside codes each
lane stores its own: the same values, bit for bit, on every tile shape, over the edges of a matrix and in front of and behind it, also in the
launch that holds both backward products, where the LDS is the larger of two products' and other workgroups take tiles of the other."""
import pytest
import torch

import paper_2403_12422_amd as jf
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


# sizes: one block, ragged tiles (blocks of 32 beyond them), several tiles each way
@pytest.mark.parametrize("block,shape", [(32, 0), (32, 1), (32, 4), (32, 6), (32, 7), (32, 8), (32, 10), (64, 1), (64, 4), (64, 11), (128, 1), (128, 6), (128, 11)])
@pytest.mark.parametrize("N,C,D", [(1, 1, 1), (3, 5, 9), (7, 11, 13)])
def test_without_codes(block, shape, N, C, D):
    N, C, D = (block * d for d in (N, C, D))
    say(f"FP32 results block {block} shape {shape} {N} x {C} -> {D}")
    g = torch.Generator(device="cuda").manual_seed(4100 + N + C + D)
    x, dy = (jf.jf_quantize_block(torch.randn((N, k), generator=g, device="cuda"), block) for k in (C, D))
    rows = torch.full((D + 64, C), 7.0, dtype=torch.float32, device="cuda")   # 32 rows of another matrix on either side
    jf.jf_debug_set_gemm_shape(shape)
    try:
        both = jf.jf_linear_wgrad(*dy, *x, block, want_q=True, want_f32=True)
        alone = jf.jf_linear_wgrad(*dy, *x, block, want_q=False, want_f32=True)
        jf.jf_linear_wgrad(*dy, *x, block, want_q=False, want_f32=True, out=(None, None, rows[32:-32]))
    finally:
        jf.jf_debug_set_gemm_shape(0)
    assert torch.equal(alone[2], both[2]) and torch.equal(rows[32:-32], both[2])
    assert bool((rows[:32] == 7.0).all()) and bool((rows[-32:] == 7.0).all())


@pytest.mark.parametrize("block,pair", [(32, p) for p in (21, 22, 23, 24, 25, 26)] + [(b, p) for b in (64, 128) for p in (21, 22, 26)])
@pytest.mark.parametrize("N,C,D", [(1, 1, 1), (7, 11, 13), (21, 13, 34)])
def test_without_codes_in_a_pair(block, pair, N, C, D):
    N, C, D = (block * d for d in (N, C, D))
    say(f"FP32 results block {block} pair {pair} {N} x {C} -> {D}")
    g = torch.Generator(device="cuda").manual_seed(4200 + N + C + D)
    x, w, dy = (jf.jf_quantize_block(torch.randn((r, k), generator=g, device="cuda"), block) for r, k in ((N, C), (D, C), (N, D)))
    dx, dw = jf.jf_linear_dgrad(*dy, *w, block), jf.jf_linear_wgrad(*dy, *x, block, want_q=True, want_f32=True)
    got = torch.empty_like(dx[0]), torch.empty_like(dx[1])
    rows = torch.full((D + 64, C), 7.0, dtype=torch.float32, device="cuda")
    jf.jf_debug_set_gemm_shape(pair)
    try:
        jf.jf_linear_bwd(*dy, *w, *x, block, out=((*got, None), (None, None, rows[32:-32])))
    finally:
        jf.jf_debug_set_gemm_shape(0)
    assert torch.equal(got[0], dx[0]) and torch.equal(got[1], dx[1])
    assert torch.equal(rows[32:-32], dw[2])
    assert bool((rows[:32] == 7.0).all()) and bool((rows[-32:] == 7.0).all())
