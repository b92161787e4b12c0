"""Outputs in the memory of inputs: what include/jetfire.h allows gives the results of separate buffers.  LayerNorm backward
takes other kernels there (other workgroups of one launch would read what it replaces); the sizes below are those where it
would otherwise run the column sums beside the rows, and those where it would not."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from paper_2403_12422_amd.build import CSRC, INCLUDE
from parity import assert_layernorm_param_grads_close
from test_gpu_parity import dev, host, say

RULE = r"""
#include "jf_common.hpp"
#include <cstdio>
int main() {
  static char m[4096];
  struct { int a, na, b, nb; bool want; } t[] = {
      {0, 64, 0, 64, true},   {0, 64, 64, 64, false}, {64, 64, 0, 64, false}, {0, 65, 64, 64, true}, {64, 64, 0, 65, true},
      {0, 4096, 100, 4, true}, {100, 4, 0, 4096, true}, {-1, 64, 0, 64, false}, {0, 64, -1, 64, false}};
  int bad = 0;
  for (auto& c : t) {
    const jf::MemRange far[] = {{m + 4000, 8}};
    const jf::MemRange a[] = {{m + 3000, 8}, {c.a < 0 ? nullptr : m + c.a, c.na}};
    const jf::MemRange b[] = {{c.b < 0 ? nullptr : m + c.b, c.nb}, {m + 3008, 8}};
    const bool whole = c.na == 4096 || c.nb == 4096;
    if (jf::any_overlap(a, b) != (c.want || whole)) ++bad;
    if (!whole && jf::any_overlap(far, b)) ++bad;
  }
  std::printf("bad %d\n", bad);
  return bad;
}
"""


def test_rule_on_memory_ranges(tmp_path):
    """Touching ranges are apart, any shared byte is not, an absent buffer shares nothing (host code, no GPU)."""
    src, exe = tmp_path / "rule.hip", tmp_path / "rule"
    src.write_text(RULE)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-w", "-I", CSRC, "-I", INCLUDE, str(src),
                    "-o", str(exe)], check=True, timeout=120)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=20)
    assert res.returncode == 0, res.stdout + res.stderr


def _same(got, want):
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("block,N,C", [(32, 96, 352), (64, 128, 192), (128, 256, 384), (32, 4096, 768)])
def test_element_wise_and_layernorm_forward(block, N, C):
    say(f"in place block={block} {N}x{C}")
    g = workloads.rng(9300 + N + C)
    (X, SX), (Z, SZ) = (tuple(map(dev, oracle.quantize_block(workloads.gaussian(g, N, C, 1.0), block))) for _ in range(2))
    gamma, beta = torch.linspace(0.5, 1.5, C, device="cuda"), torch.linspace(-0.1, 0.1, C, device="cuda")
    mask = dev(g.integers(0, 256, (N, C // 8), dtype=np.uint8))
    mean, rstd = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
    ops = {
        "gelu": lambda a, b, out: jf.jf_gelu_q(*a, block, out=out),
        "gelu backward": lambda a, b, out: jf.jf_gelu_q_bwd(*a, *b, block, out=out),
        "add": lambda a, b, out: jf.jf_add_q(*a, *b, block, out=out),
        "dropout": lambda a, b, out: jf.jf_dropout_q(*a, mask, 0.25, block, out=out),
        "layernorm": lambda a, b, out: jf.jf_layernorm_q(*a, gamma, beta, 1e-5, block, out=out and (*out, mean, rstd)),
    }
    for name, op in ops.items():
        want = op((X, SX), (Z, SZ), None)[:2]
        for first in (True, False)[: 2 if name in ("gelu backward", "add") else 1]:
            say(f"  {name}, over the {'first' if first else 'second'} operand")
            a, b = (X.clone(), SX.clone()), (Z.clone(), SZ.clone())
            _same(op(a, b, a if first else b)[:2], want)


@pytest.mark.gpu
@pytest.mark.parametrize("block,N,C", [(32, 32, 32), (32, 384, 128), (32, 768, 160), (32, 1024, 2048), (32, 2048, 704), (32, 2080, 704),
                                       (32, 96, 2080), (64, 1088, 320), (128, 384, 1152)])
def test_layernorm_backward(block, N, C):
    say(f"layernorm backward in place block={block} {N}x{C}")
    g = workloads.rng(9400 + N + C)
    X, SX = oracle.quantize_block(workloads.gaussian(g, N, C, 1.0), block)
    G, SG = oracle.quantize_block(workloads.gaussian(g, N, C, 1e-3), block)
    gamma = (1.0 + 0.1 * g.standard_normal(C, dtype=np.float32)).astype(np.float32)
    mean, rstd = oracle.layernorm_q(X, SX, gamma, np.zeros(C, np.float32), 1e-5, block)[2:4]
    o = oracle.layernorm_q_bwd(G, SG, X, SX, gamma, mean, rstd, block)
    xh = (oracle.dequantize(X, SX, block) - mean[:, None].astype(np.float64)) * rstd[:, None].astype(np.float64)
    want = jf.jf_layernorm_q_bwd(*map(dev, (G, SG, X, SX, gamma, mean, rstd)), block)
    for over in ("dY", "X", "dY and gamma", "gamma"):
        say(f"  over {over}")
        t = dict(zip(("dY", "SdY", "X", "SX", "gamma", "mean", "rstd"), map(dev, (G, SG, X, SX, gamma, mean, rstd))))
        q = over.split()[0]
        out = [t[q], t["S" + q]] if q != "gamma" else [torch.empty_like(t["X"]), torch.empty_like(t["SX"])]
        out += [t["gamma"] if "gamma" in over else torch.empty_like(t["gamma"]), torch.empty_like(t["gamma"])]
        dX, SdX, dg, db = jf.jf_layernorm_q_bwd(*t.values(), block, out=tuple(out))
        _same((dX, SdX), want[:2])
        assert_layernorm_param_grads_close(host(dg), host(db), o[2], o[3], oracle.dequantize(G, SG, block), xh, over)


@pytest.mark.gpu
@pytest.mark.parametrize("block", [32, 64, 128])
@pytest.mark.parametrize("blocks", [(3, 5, 2), (8, 8, 8), (37, 5, 3)])
def test_weight_gradient_over_the_weights(block, blocks):
    N, C, D = (block * b for b in blocks)
    g = workloads.rng(9500 + N)
    quantized = lambda r, c, std: tuple(map(dev, oracle.quantize_block(workloads.gaussian(g, r, c, std), block)))
    X, W, dY = quantized(N, C, 1.0), quantized(D, C, 0.02), quantized(N, D, 1e-3)
    want = jf.jf_linear_dgrad(*dY, *W, block), jf.jf_linear_wgrad(*dY, *X, block)
    try:
        for shape in (0, 21, 22):   # automatic, and both products asked for in one launch
            say(f"weight gradient over the weights block={block} {N} x {C} -> {D}, shape {shape}")
            jf.jf_debug_set_gemm_shape(shape)
            Wc = tuple(t.clone() for t in W)
            dX = torch.empty((N, C), dtype=torch.int8, device="cuda"), torch.empty((N // block, C // block), device="cuda")
            got = jf.jf_linear_bwd(*dY, *Wc, *X, block, out=((*dX, None), (*Wc, None)))
            _same(got[0][:2], want[0][:2])
            _same(got[1][:2], want[1][:2])
    finally:
        jf.jf_debug_set_gemm_shape(0)
