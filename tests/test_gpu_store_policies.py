"""Operators whose results are stored in another way from some size on: a large tensor against the same rows in calls that
are too small for that (every block is computed by itself, so all results are equal bit for bit; run with -m gpu)."""
import pytest
import torch

import paper_2403_12422_amd as jf
from test_gpu_parity import say

pytestmark = pytest.mark.gpu
# just past 64 MB in whole lines, just past 32 MB in rows that share lines; small calls of 128 rows and of 1/8
SIZES = [(32, 87424, 768), (64, 87424, 768), (128, 87424, 768), (32, 42112, 800), (64, 40448, 832)]


def _tensor(g, n, c, block):
    return (torch.randint(-127, 128, (n, c), dtype=torch.int8, device="cuda", generator=g),
            0.01 + torch.rand((n // block, c // block), device="cuda", generator=g))


@pytest.mark.parametrize("block,N,C", SIZES)
def test_large_results_equal_those_of_small_calls(block, N, C):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + C + block)
    (X, SX), (Z, SZ) = _tensor(g, N, C, block), _tensor(g, N, C, block)
    mask = torch.randint(0, 256, (N, C // 8), dtype=torch.uint8, device="cuda", generator=g)
    x32 = torch.randn((N, C), device="cuda", generator=g)
    ops = {
        "add": lambda r, b: jf.jf_add_q(X[r], SX[b], Z[r], SZ[b], block),
        "add with row partials": lambda r, b: jf.jf_add_q(X[r], SX[b], Z[r], SZ[b], block, want_partials=True),
        "gelu": lambda r, b: jf.jf_gelu_q(X[r], SX[b], block),
        "gelu backward": lambda r, b: jf.jf_gelu_q_bwd(Z[r], SZ[b], X[r], SX[b], block),
        "dropout": lambda r, b: jf.jf_dropout_q(X[r], SX[b], mask[r], 0.25, block),
        "quantize FP32": lambda r, b: jf.jf_quantize_block(x32[r], block),
        "quantize FP16": lambda r, b: jf.jf_quantize_block(x32[r].half(), block),
    }
    whole = slice(None)
    parts = [(0, 128), (128, N // 8 // 128 * 128), (N - 128, N)]
    for name, op in ops.items():
        say(f"{name} block={block} {N} x {C}")
        got = op(whole, whole)
        for first, last in parts:
            rows, brows = slice(first, last), slice(first // block, last // block)
            want = op(rows, brows)
            assert torch.equal(got[0][rows], want[0]), name
            assert torch.equal(got[1][brows], want[1]), name
            for a, b in zip(got[2:], want[2:]):   # row partials: block column by block column
                assert torch.equal(a[:, rows], b), name


# 5, 6 and 9 strips of 128 columns: FP16 by one, by two, and by two with none in the last place; rows that end amid a tile of 128
@pytest.mark.parametrize("block", [32, 64, 128])
@pytest.mark.parametrize("N,C", [(104960, 640), (87424, 768), (58368, 1152)])
def test_streamed_quantizer(block, N, C):
    if block == 32:
        N += 32
    g = torch.Generator(device="cuda")
    g.manual_seed(N + C + block)
    x32 = torch.randn((N, C), device="cuda", generator=g)
    for x in (x32, x32.half()):
        say(f"streamed quantizer {x.dtype} block={block} {N} x {C}")
        q, s = jf.jf_quantize_block(x, block)
        qt = jf.jf_quantize_block(x, block, transposed_copy=True)
        assert torch.equal(qt[0], q) and torch.equal(qt[1], s)
        assert torch.equal(qt[2], q.t()) and torch.equal(qt[3], s.t())
        part = 12800
        for first in range(0, N, part):
            rows, brows = slice(first, min(first + part, N)), slice(first // block, min(first + part, N) // block)
            want = jf.jf_quantize_block(x[rows], block)
            assert torch.equal(q[rows], want[0]) and torch.equal(s[brows], want[1])


# FP32 with the transposed copy from 22 M elements on, written through, written back, written through: fewer workgroups on a compute unit
@pytest.mark.parametrize("block,N,C", [(32, 22112, 1024), (64, 16448, 2112), (128, 32896, 768)])
def test_large_transposed_copy(block, N, C):
    say(f"large transposed copy block={block} {N} x {C}")
    assert N * C >= 21 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(N + C + block)
    x = torch.randn((N, C), device="cuda", generator=g)
    q, s, qT, sT = jf.jf_quantize_block(x, block, transposed_copy=True)
    assert torch.equal(qT, q.t()) and torch.equal(sT, s.t())
    part = 4096
    for first in range(0, N, part):
        rows, brows = slice(first, min(first + part, N)), slice(first // block, min(first + part, N) // block)
        want = jf.jf_quantize_block(x[rows], block)
        assert torch.equal(q[rows], want[0]) and torch.equal(s[brows], want[1])


# FP32 from 335 M elements on, in whole lines and in rows that share them: another number of chunks a thread
@pytest.mark.parametrize("block,N,C", [(32, 87392, 3840), (64, 419456, 800 + 32), (128, 65664, 5120)])
def test_large_dequantizer(block, N, C):
    say(f"large dequantizer block={block} {N} x {C}")
    assert N * C >= 320 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(N + C)
    X, SX = _tensor(g, N, C, block)
    got = jf.jf_dequantize_block(X, SX, block, torch.float32)
    part = N // 16 // 128 * 128
    for first in range(0, N, part):
        rows, brows = slice(first, min(first + part, N)), slice(first // block, min(first + part, N) // block)
        assert torch.equal(got[rows], jf.jf_dequantize_block(X[rows], SX[brows], block, torch.float32))
