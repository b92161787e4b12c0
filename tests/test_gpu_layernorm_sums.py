"""The two-kernel LayerNorm backward and the row statistics from an Add's partials: column ranges of unequal ends, one to sixteen waves of
strips, row blocks requested ahead (four or more to a workgroup) and not."""
import pytest

import test_gpu_layernorm_block_rows as block_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,N,C", [(32, 32, 2080), (32, 96, 4224), (32, 256, 6176), (64, 64, 1088), (64, 192, 2112), (64, 66304, 1088), (128, 128, 640),
                                       (128, 384, 2176), (128, 66560, 640)])
def test_layernorm_sums(block, N, C):
    block_rows.test_layernorm_block_rows(block, N, C)
