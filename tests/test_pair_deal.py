"""How the tiles of both backward products are dealt to the workgroups of one launch: every tile once, on its XCD, and on a compute unit no
more than in order (host code); and the products that come out of it (on the GPU)."""
import os
import subprocess

import pytest
import torch

import paper_2403_12422_amd as jf
from paper_2403_12422_amd.build import CSRC, INCLUDE
from test_gpu_parity import say

DEAL = r"""
#include "jf_gemm_kernel.hpp"
#include <cstdio>
#include <vector>
int main() {
  long bad = 0, dealt = 0;
  for (int resident = 2; resident <= 4; ++resident)
    for (int first = 1; first < 900; first += first < 20 ? 1 : 13)
      for (int second = 1; second < 900; second += second < 20 ? 1 : 11)
        for (double work : {1.0, 1.33, 4.0}) {
          double most = 0;
          const jf::PairDeal d = jf::deal_pair(first, second, work, 1.0, resident, &most);
          const jf::PairDeal plain = {d.split, 0, 0, 0};
          const int all = d.split + ((second + 7) & ~7);
          std::vector<int> seen(all);
          std::vector<double> load(256), in_order(256);
          for (int i = 0; i < all; ++i) {
            int tile = -1;
            const bool early = d.place(i, tile);
            if (tile < 0 || tile >= (early ? d.split : all - d.split) || tile % 8 != i % 8) ++bad;
            else ++seen[early ? tile : d.split + tile];
            load[i % 256] += early ? work : 1.0;
            in_order[i % 256] += plain.place(i, tile) ? work : 1.0;
          }
          for (int n : seen) bad += n != 1;
          const double a = *std::max_element(load.begin(), load.end()), b = *std::max_element(in_order.begin(), in_order.end());
          if (a > b + 1e-9 || (d.few && (a > most + 1e-9 || all <= 256 || all > 256 * resident))) ++bad;
          dealt += d.few > 0;
        }
  std::printf("bad %ld dealt %ld\n", bad, dealt);
  return bad != 0 || dealt < 1000;
}
"""


def test_every_tile_once(tmp_path):
    src, exe = tmp_path / "deal.hip", tmp_path / "deal"
    src.write_text(DEAL)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", CSRC, "-I", INCLUDE, str(src),
                    "-o", str(exe)], check=True, timeout=120)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr


# tiles by turns of 256 with a rest: two and three on a unit, the longer ones in either product
@pytest.mark.gpu
@pytest.mark.parametrize("pair,N,C,D", [(26, 4096, 768, 3072), (26, 1472, 928, 2208), (23, 1056, 800, 2080), (23, 1472, 928, 2208), (22, 2304, 1408, 1952),
                                        (21, 3072, 2048, 3168), (24, 416, 1120, 2208), (25, 2208, 1120, 416)])
def test_products(pair, N, C, D):
    say(f"pair {pair} {N} x {C} -> {D}")
    g = torch.Generator(device="cuda").manual_seed(7700 + N + C + D)
    x, w, dy = (jf.jf_quantize_block(torch.randn((r, c), generator=g, device="cuda"), 32) for r, c in ((N, C), (D, C), (N, D)))
    want = jf.jf_linear_dgrad(*dy, *w, 32), jf.jf_linear_wgrad(*dy, *x, 32)
    jf.jf_debug_set_gemm_shape(pair)
    try:
        got = jf.jf_linear_bwd(*dy, *w, *x, 32)
    finally:
        jf.jf_debug_set_gemm_shape(0)
    for a, b in zip(got, want):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
