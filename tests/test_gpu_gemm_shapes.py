"""GPU parity of the block-32 32x32 tile, of contraction lengths beyond one segment of 64 block scales, and of the two backward
products in one launch."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from test_gpu_parity import _k_sweep_case, _quantized_layer, dev, host, say

pytestmark = pytest.mark.gpu
SHAPES = {32: (1, 4, 6, 8, 10), 64: (1, 4), 128: (1, 6)}
PAIRS = {32: (21, 22, 23, 24, 25), 64: (21, 22), 128: (21, 22)}


@pytest.fixture
def forced():
    yield jf.jf_debug_set_gemm_shape
    jf.jf_debug_set_gemm_shape(0)


def _same(got, want):
    for a, b in zip(got, want):
        np.testing.assert_array_equal(host(a), b)


def test_fine_tile_every_stage_count(forced):
    forced(10)
    for nsteps in list(range(1, 19)) + [31, 33, 47]:
        say(f"32x32 tile: {nsteps} K steps")
        (X, SX, W, SW, dY, SdY), f_fwd, f_dgrad, f_wgrad = _k_sweep_case(nsteps)
        Xd, SXd, Wd, SWd, dYd, SdYd = map(dev, (X, SX, W, SW, dY, SdY))
        np.testing.assert_array_equal(host(jf.jf_linear_fwd(Xd, SXd, Wd, SWd, 32, want_f32=True)[2]), f_fwd)
        np.testing.assert_array_equal(host(jf.jf_linear_dgrad(dYd, SdYd, Wd, SWd, 32, want_f32=True)[2]), f_dgrad)
        np.testing.assert_array_equal(host(jf.jf_linear_wgrad(dYd, SdYd, Xd, SXd, 32, want_f32=True)[2]), f_wgrad)


@pytest.mark.parametrize("block", [32, 64, 128])
def test_more_k_blocks_than_a_segment_of_scales(block, forced):
    for nkb in (59, 60, 61, 63, 64, 65, 120, 121, 131):
        k, n = block * nkb, 2 * block
        for axis, dims in enumerate(((n, k, n), (n, n, k), (k, n, n))):   # the contraction length of forward, dgrad, wgrad
            (X, SX), (W, SW), (dY, SdY) = _quantized_layer(5200 + nkb + axis, *dims, block)
            Xd, SXd, Wd, SWd, dYd, SdYd = map(dev, (X, SX, W, SW, dY, SdY))
            want = (oracle.linear_fwd(X, SX, W, SW, block), oracle.linear_dgrad(dY, SdY, W, SW, block),
                    oracle.linear_wgrad(dY, SdY, X, SX, block))[axis]
            for shape in SHAPES[block]:
                say(f"block {block} shape {shape} axis {axis}: {nkb} K blocks")
                forced(shape)
                got = (lambda: jf.jf_linear_fwd(Xd, SXd, Wd, SWd, block, want_f32=True),
                       lambda: jf.jf_linear_dgrad(dYd, SdYd, Wd, SWd, block, want_f32=True),
                       lambda: jf.jf_linear_wgrad(dYd, SdYd, Xd, SXd, block, want_f32=True))[axis]()
                _same(got, want[:3])


@pytest.mark.parametrize("block", [32, 64, 128])
@pytest.mark.parametrize("blocks", [(1, 1, 1), (3, 5, 2), (9, 2, 7), (2, 11, 13), (37, 5, 3)])
def test_backward_products_in_one_launch(block, blocks, forced):
    N, C, D = (block * b for b in blocks)
    (X, SX), (W, SW), (dY, SdY) = _quantized_layer(5600 + sum(blocks), N, C, D, block)
    Xd, SXd, Wd, SWd, dYd, SdYd = map(dev, (X, SX, W, SW, dY, SdY))
    want = oracle.linear_dgrad(dY, SdY, W, SW, block)[:3], oracle.linear_wgrad(dY, SdY, X, SX, block)[:3]
    for pair in (0,) + PAIRS[block]:
        say(f"block {block} pair {pair}: {N} x {C} -> {D}")
        forced(pair)
        for got, w in zip(jf.jf_linear_bwd(dYd, SdYd, Wd, SWd, Xd, SXd, block, want_f32=True), want):
            _same(got, w)
