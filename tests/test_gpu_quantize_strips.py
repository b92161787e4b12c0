"""The quantizer on strips of 64 and 128 columns: sizes on both sides of the line between them, with ragged last tiles, against
the oracle (codes and scales are exact)."""
import numpy as np
import pytest

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("block,rows,cols", [
    (32, 96, 224), (32, 1024, 1024), (32, 1056, 1056), (32, 2048, 2080), (32, 2048, 6144), (32, 2080, 6176),
    (64, 64, 64), (64, 1088, 960), (64, 2048, 2048), (64, 2048, 2112), (64, 2112, 6208),
    (128, 128, 128), (128, 1152, 896), (128, 2048, 2048), (128, 2176, 2048), (128, 3072, 4224)])
def test_quantize_strips(block, rows, cols, dtype):
    say(f"quantize strips block={block} {rows}x{cols} {dtype}")
    g = workloads.rng(9700 + block + rows + cols)
    x = workloads.gaussian(g, rows, cols, 1.0)
    x[-1, :] *= 30.0                                          # every block's largest element beside its neighbours' in a corner
    x[:, -1] *= 50.0
    x = x.astype(np.float16).astype(np.float32)
    oq, os_ = oracle.quantize_block(x, block)
    q, s = jf.jf_quantize_block(dev(x if dtype == "f32" else x.astype(np.float16)), block)
    np.testing.assert_array_equal(host(s), os_)
    np.testing.assert_array_equal(host(q), oq)
