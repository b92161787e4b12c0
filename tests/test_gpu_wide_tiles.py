"""GPU parity of the persistent 256x256 tile (block sizes 64 and 128): against the oracle where a workgroup has one tile, and
against the other tile shapes, bit for bit, where it goes on to a second one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_12422_amd as jf
from test_gpu_parity import _quantized_layer, dev, host, say

pytestmark = pytest.mark.gpu
WIDE, WIDE_PAIR = 11, 26


@pytest.fixture
def forced():
    yield jf.jf_debug_set_gemm_shape
    jf.jf_debug_set_gemm_shape(0)


def _products(layer, block, f32=True):
    (x, sx), (w, sw), (dy, sdy) = layer
    return (jf.jf_linear_fwd(x, sx, w, sw, block, want_f32=f32), jf.jf_linear_dgrad(dy, sdy, w, sw, block, want_f32=f32),
            jf.jf_linear_wgrad(dy, sdy, x, sx, block, want_f32=f32))


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("blocks", [(1, 1, 1), (2, 3, 4), (5, 1, 3), (3, 9, 2), (4, 2, 66), (65, 3, 1), (7, 64, 5)])
def test_against_the_oracle(block, blocks, forced):
    """Ragged tiles in both directions and every contraction length modulo the ring, beyond 64 K blocks as well."""
    N, C, D = (block * b for b in blocks)
    say(f"256x256 tile block={block} {N} x {C} -> {D}")
    (X, SX), (W, SW), (dY, SdY) = _quantized_layer(7100 + block + sum(blocks), N, C, D, block)
    layer = (dev(X), dev(SX)), (dev(W), dev(SW)), (dev(dY), dev(SdY))
    want = (oracle.linear_fwd(X, SX, W, SW, block), oracle.linear_dgrad(dY, SdY, W, SW, block), oracle.linear_wgrad(dY, SdY, X, SX, block))
    forced(WIDE)
    for got, w in zip(_products(layer, block), want):
        for a, b in zip(got, w[:3]):
            np.testing.assert_array_equal(host(a), b)
    q, s, f = jf.jf_linear_wgrad(*layer[2], *layer[0], block, want_q=False, want_f32=True)
    assert q is None and s is None
    np.testing.assert_array_equal(host(f), want[2][2])
    forced(WIDE_PAIR)
    for got, w in zip(jf.jf_linear_bwd(*layer[2], *layer[1], *layer[0], block, want_f32=True), want[1:]):
        for a, b in zip(got, w[:3]):
            np.testing.assert_array_equal(host(a), b)


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("kblocks", [1, 2, 3, 4, 5, 9])
def test_from_tile_to_tile(block, kblocks, forced):
    """Outputs of 17 x 17 tiles, the last ones ragged: 33 workgroups take a second tile, which begins at every place of the ring."""
    m, n, k = 17 * 256 - block, 16 * 256 + block, kblocks * block
    g = torch.Generator(device="cuda").manual_seed(7300 + block + kblocks)
    draw = lambda r, c: jf.jf_quantize_block(torch.randn((r, c), generator=g, device="cuda"), block)
    for which, (N, C, D) in enumerate(((m, k, n), (m, n, k), (k, n, m))):   # forward, input gradient, weight gradient
        say(f"256x256 tile block={block} product {which}: {kblocks} K blocks")
        layer = draw(N, C), draw(D, C), draw(N, D)
        forced(1)
        want = _products(layer, block)[which]
        forced(WIDE)
        for a, b in zip(_products(layer, block)[which], want):
            assert torch.equal(a, b)


@pytest.mark.parametrize("tiles", [(12, 17), (41, 5), (14, 15), (25, 20)])
@pytest.mark.parametrize("kblocks", [1, 2, 3, 4, 5, 9])
def test_quarters_and_whole_sub_blocks(tiles, kblocks, forced):
    """Either side of the number of tiles from which on sub-blocks are multiplied in quarters (204 and 205), and two tiles to a workgroup so, the
    last ones of a row and a column ragged."""
    block, m, n, k = 128, tiles[0] * 256 - 128, tiles[1] * 256 - 128, kblocks * 128
    g = torch.Generator(device="cuda").manual_seed(7400 + tiles[0] + kblocks)
    draw = lambda r, c: jf.jf_quantize_block(torch.randn((r, c), generator=g, device="cuda"), block)
    say(f"256x256 tiles {tiles} {kblocks} K blocks")
    (a, sa), fwd_w, dgrad_w = draw(m, k), draw(n, k), draw(k, n)
    both = lambda: (jf.jf_linear_fwd(a, sa, *fwd_w, block, want_f32=True), jf.jf_linear_dgrad(a, sa, *dgrad_w, block, want_f32=True))
    forced(1)
    want = both()
    forced(WIDE)
    for got, ref in zip(both(), want):
        for x, y in zip(got, ref):
            assert torch.equal(x, y)


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("sizes", [(2816, 4352, 1408), (1408, 4352, 2816), (5120, 4096, 4352)])
def test_both_backward_products_as_one_list(block, sizes, forced):
    """One list of tiles: workgroups with tiles of both products, of one only and with several of each; either product first."""
    N, C, D = sizes
    g = torch.Generator(device="cuda").manual_seed(7500 + block + N)
    draw = lambda r, c: jf.jf_quantize_block(torch.randn((r, c), generator=g, device="cuda"), block)
    x, w, dy = draw(N, C), draw(D, C), draw(N, D)
    say(f"256x256 pair block={block} {N} x {C} -> {D}")
    forced(1)
    want = jf.jf_linear_dgrad(*dy, *w, block), jf.jf_linear_wgrad(*dy, *x, block)
    forced(WIDE_PAIR)
    for _ in range(2):
        for got, ref in zip(jf.jf_linear_bwd(*dy, *w, *x, block), want):
            for a, b in zip(got[:2], ref[:2]):
                assert torch.equal(a, b)
