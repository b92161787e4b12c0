"""GPU parity of the block-32 128x64 tile of eight waves and of its pair of backward products: every number of stages, more K blocks than a
segment of scales, ragged tiles in both directions."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from test_gpu_parity import _k_sweep_case, _quantized_layer, dev, host, say
from test_gpu_wide_tiles import _products, forced   # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu
SHAPE, PAIR = 7, 26


def test_every_stage_count(forced):   # noqa: F811
    forced(SHAPE)
    for nsteps in list(range(1, 14)) + [31, 33, 47]:
        say(f"128x64 tile of eight waves: {nsteps} K steps")
        (X, SX, W, SW, dY, SdY), f_fwd, f_dgrad, f_wgrad = _k_sweep_case(nsteps)
        Xd, SXd, Wd, SWd, dYd, SdYd = map(dev, (X, SX, W, SW, dY, SdY))
        np.testing.assert_array_equal(host(jf.jf_linear_fwd(Xd, SXd, Wd, SWd, 32, want_f32=True)[2]), f_fwd)
        np.testing.assert_array_equal(host(jf.jf_linear_dgrad(dYd, SdYd, Wd, SWd, 32, want_f32=True)[2]), f_dgrad)
        np.testing.assert_array_equal(host(jf.jf_linear_wgrad(dYd, SdYd, Xd, SXd, 32, want_f32=True)[2]), f_wgrad)


@pytest.mark.parametrize("N,C,D", [(32, 32, 32), (128, 64, 128), (160, 96, 224), (2080, 65 * 32, 96), (64 * 32, 288, 352), (131 * 32, 64, 160)])
def test_against_the_oracle(N, C, D, forced):   # noqa: F811
    say(f"128x64 tile of eight waves {N} x {C} -> {D}")
    (X, SX), (W, SW), (dY, SdY) = _quantized_layer(7600 + N + C + D, N, C, D, 32)
    layer = (dev(X), dev(SX)), (dev(W), dev(SW)), (dev(dY), dev(SdY))
    want = (oracle.linear_fwd(X, SX, W, SW, 32), oracle.linear_dgrad(dY, SdY, W, SW, 32), oracle.linear_wgrad(dY, SdY, X, SX, 32))
    forced(SHAPE)
    for got, w in zip(_products(layer, 32), want):
        for a, b in zip(got, w[:3]):
            np.testing.assert_array_equal(host(a), b)
    forced(PAIR)
    for got, w in zip(jf.jf_linear_bwd(*layer[2], *layer[1], *layer[0], 32, want_f32=True), want[1:]):
        for a, b in zip(got, w[:3]):
            np.testing.assert_array_equal(host(a), b)
