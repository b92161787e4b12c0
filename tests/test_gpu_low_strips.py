"""GELU, Add and Dropout of small tensors in waves of 16 rows: a last strip with one block, a last workgroup with strips that do not exist
(against the oracle), and sizes up to and behind the lines to waves of 32 rows (against their small calls, bit for bit)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_12422_amd as jf
import test_gpu_store_policies as policies
import test_gpu_strips as strips
from paper_2403_12422_amd import workloads
from test_gpu_parity import _check_eltwise, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,N,C", [(32, 2176, 992), (32, 9856, 1280), (64, 2176, 1024), (64, 9856, 1280), (128, 13184, 1280), (128, 26368, 1280),
                                       (32, 14720, 1280), (32, 14752, 1280), (64, 10944, 1152), (64, 40256, 832),
                                       (32, 3296, 1280), (32, 10656, 1280), (32, 11520, 1280), (64, 9088, 1280)])
def test_behind_the_lines(block, N, C):
    policies.test_large_results_equal_those_of_small_calls(block, N, C)


@pytest.mark.parametrize("block,N,C", [(32, 32, 32), (32, 96, 160), (32, 160, 448), (32, 8192, 1280), (64, 64, 64), (64, 192, 320), (128, 128, 128),
                                       (128, 384, 640)])
def test_low_strips(block, N, C):
    strips.test_workgroups_of_four_waves(block, N, C)
    g = workloads.rng(9800 + N + C)
    X, SX = oracle.quantize_block(workloads.gaussian(g, N, C, 2.0), block)
    Z, SZ = oracle.quantize_block(workloads.gaussian(g, N, C, 1.0), block)
    o = oracle.add_q(X, SX, Z, SZ, block)
    mask = torch.randint(0, 256, (N, C // 8), dtype=torch.uint8, device="cuda")
    od = oracle.dropout_q(X, SX, host(mask), 0.25, block)
    _check_eltwise("dropout", *jf.jf_dropout_q(dev(X), dev(SX), mask, 0.25, block), *od[:2], od[2], block)
    plain = jf.jf_add_q(*map(dev, (X, SX, Z, SZ)), block)
    q, s, mean, sumsq = jf.jf_add_q(*map(dev, (X, SX, Z, SZ)), block, want_partials=True)
    assert torch.equal(q, plain[0]) and torch.equal(s, plain[1])
    _check_eltwise("add", q, s, *o[:2], o[4], block)
    y = o[4].reshape(N, C // block, block)
    say("  row partials")   # 32-bit terms and sums: less than 2 B roundings of 2^-24 each, against magnitudes
    tol = 2 * block * 2.0 ** -24
    assert np.all(np.abs(host(mean) - y.mean(2).T) <= tol * np.abs(y).mean(2).T)
    assert np.all(np.abs(host(sumsq) - (y * y).sum(2).T) <= tol * (y * y).sum(2).T + 1e-30)
