"""GELU and Add of small tensors on strips of 64 columns: a last strip with one block or none, a last workgroup with strips that do not
exist (against the oracle), and sizes behind the lines to strips of 128 columns (against their small calls, bit for bit)."""
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


@pytest.mark.parametrize("block,N,C", [(32, 8320, 1280), (32, 19712, 1280), (32, 26368, 1280), (64, 8320, 1280), (64, 9856, 1280)])
def test_behind_the_lines(block, N, C):
    policies.test_large_results_equal_those_of_small_calls(block, N, C)


@pytest.mark.parametrize("block,N,C", [(32, 32, 32), (32, 96, 160), (32, 160, 448), (32, 8192, 1280), (64, 64, 64), (64, 192, 320)])
def test_narrow_strips(block, N, C):
    strips.test_workgroups_of_four_waves(block, N, C)
    g = workloads.rng(9800 + N + C)
    X, SX = oracle.quantize_block(workloads.gaussian(g, N, C, 2.0), block)
    Z, SZ = oracle.quantize_block(workloads.gaussian(g, N, C, 1.0), block)
    o = oracle.add_q(X, SX, Z, SZ, block)
    plain = jf.jf_add_q(*map(dev, (X, SX, Z, SZ)), block)
    q, s, mean, sumsq = jf.jf_add_q(*map(dev, (X, SX, Z, SZ)), block, want_partials=True)
    assert torch.equal(q, plain[0]) and torch.equal(s, plain[1])
    _check_eltwise("add", q, s, *o[:2], o[4], block)
    y = o[4].reshape(N, C // block, block)
    say("  row partials")   # 32-bit terms and sums: less than 2 B roundings of 2^-24 each, against magnitudes
    tol = 2 * block * 2.0 ** -24
    assert np.all(np.abs(host(mean) - y.mean(2).T) <= tol * np.abs(y).mean(2).T)
    assert np.all(np.abs(host(sumsq) - (y * y).sum(2).T) <= tol * (y * y).sum(2).T + 1e-30)
