"""The products on the shapes that the model picks, against one forced shape, bit for bit: layers in whole rounds of tiles, a little more
than a round, operands beyond the caches, and layers where the two backward products go in one launch and in two."""
import pytest
import torch

import paper_2403_12422_amd as jf
from test_gpu_parity import say
from test_gpu_wide_tiles import _products, forced   # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,N,C,D", [(32, 2048, 2048, 2048), (32, 2560, 2560, 3072), (32, 5120, 1280, 5120), (32, 8192, 8192, 4096), (32, 2112, 1760, 9824),
                                         (32, 512, 8192, 8192), (64, 1536, 5120, 3072), (64, 5120, 1024, 1536), (128, 2048, 3072, 4096), (128, 512, 7296, 128)])
def test_chosen_shapes(block, N, C, D, forced):   # noqa: F811
    say(f"chosen shapes block={block} {N} x {C} -> {D}")
    g = torch.Generator(device="cuda").manual_seed(7500 + N + C + D)
    layer = [jf.jf_quantize_block(torch.randn((r, c), generator=g, device="cuda"), block) for r, c in ((N, C), (D, C), (N, D))]
    forced(1)
    want = _products(layer, block, f32=False)
    forced(0)
    got = _products(layer, block, f32=False)
    pair = jf.jf_linear_bwd(*layer[2], *layer[1], *layer[0], block)
    for a, b in zip(got + tuple(pair), want + want[1:]):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
