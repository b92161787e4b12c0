"""Element-wise operators at block sizes 64 and 128 on strips: a last workgroup of eight waves with strips that do not exist (against
small calls, bit for bit), and the smallest and ragged tensors in workgroups of one block row (against the oracle)."""
import pytest

import oracle
import paper_2403_12422_amd as jf
import test_gpu_store_policies as policies
from paper_2403_12422_amd import workloads
from test_gpu_parity import _check_eltwise, dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,N,C", [(64, 40512, 832), (128, 75136, 896)])
def test_workgroups_of_eight_waves(block, N, C):
    policies.test_large_results_equal_those_of_small_calls(block, N, C)


@pytest.mark.parametrize("block,N,C", [(64, 192, 64), (64, 64, 320), (128, 128, 128), (128, 384, 640)])
def test_workgroups_of_four_waves(block, N, C):
    say(f"strips block={block} {N} x {C}")
    g = workloads.rng(9600 + N + C)
    X, SX = oracle.quantize_block(workloads.gaussian(g, N, C, 2.0), block)
    G, SG = oracle.quantize_block(workloads.gaussian(g, N, C, 1e-3), block)
    args = dev(X), dev(SX), dev(G), dev(SG)
    o = oracle.gelu_q(X, SX, block)
    _check_eltwise("gelu", *jf.jf_gelu_q(*args[:2], block), *o[:2], o[2], block)
    o = oracle.gelu_q_bwd(G, SG, X, SX, block)
    _check_eltwise("gelu backward", *jf.jf_gelu_q_bwd(*args[2:], *args[:2], block), *o[:2], o[2], block)
