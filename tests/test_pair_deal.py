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


# jf_linear_bwd itself, with the launches recorded instead of made: the deal that is launched against the one that the choice counts on
LAUNCHED = r"""
#include "jf_common.hpp"
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(KERNEL, GRID, BLOCK, LDS, STREAM, ...) record(GRID, __VA_ARGS__)
struct { int pairs = 0, grid = 0, second_first = 0, deal[4] = {}; } seen;
template <class... REST> void record(dim3, REST...) {}   // other kernels
template <class A, class... REST> void record(dim3 grid, A, jf::v4i sizes, jf::v4i deal, REST...) {
  seen.pairs += 1, seen.grid = (int)grid.x, seen.second_first = sizes[3];
  for (int i = 0; i < 4; ++i) seen.deal[i] = deal[i];
}
#include "jf_gemm_fine.hpp"
#include "jf_gemm_wide.hpp"
#include "jf_gemm_bwd_pair_b32.hip"
#include "jf_gemm_bwd_pair_b64.hip"
#include "jf_gemm_bwd_pair_b128.hip"
#include "jf_linear.hip"
#include <cstdio>
#include <random>
#include <vector>
namespace jf {
thread_local int32_t g_last_hip_error = 0;
#define ONE_PRODUCT(B) void launch_gemm_fwd_b##B(int, const GemmArgs&, bool, hipStream_t) {} \
  void launch_gemm_dgrad_b##B(int, const GemmArgs&, bool, hipStream_t) {} void launch_gemm_wgrad_b##B(int, const GemmArgs&, bool, hipStream_t) {}
ONE_PRODUCT(32) ONE_PRODUCT(64) ONE_PRODUCT(128)
}
using namespace jf;
int main() {
  std::mt19937 rng(5);
  const auto size = [&](int b, double lo, double hi) {
    return (int64_t)b * std::max(1, (int)std::lround(std::exp(std::uniform_real_distribution<double>(std::log(lo), std::log(hi))(rng)) / b));
  };
  long worse = 0, unforeseen = 0, launched = 0, dealt = 0;
  for (int layer = 0; layer < 6000; ++layer) {
    const int b = layer % 4 < 2 ? 32 : layer % 4 == 2 ? 64 : 128;
    const int64_t N = size(b, 128, 16384), C = size(b, 128, 6144), D = size(b, 128, 6144);
    const ShapeTable t = shape_table(b);
    GemmArgs d{}, w{};
    d.M = (int)N, d.Nn = (int)C, d.K = (int)D, w.M = (int)D, w.Nn = (int)C, w.K = (int)N;
    const int chosen = choose_pair(b, d, w, 0).pair;
    for (int i = -1; i < t.npairs; ++i) {   // the pair that is chosen, then each of them
      const int pair = i < 0 ? chosen : t.pairs[i].pair;
      if (pair == 0) continue;
      const PairModel& p = *std::find_if(t.pairs, t.pairs + t.npairs, [&](const PairModel& m) { return m.pair == pair; });
      const ShapeModel &sd = *t.find(p.dgrad), &sw = *t.find(p.wgrad);
      if (sd.resident == kPersistent) continue;
      int8_t* const q = (int8_t*)((size_t)1 << 40);   // never read
      float* const s = (float*)((size_t)1 << 41);
      const size_t far = (size_t)1 << 34;
      seen.pairs = 0;
      jf_debug_set_gemm_shape(i < 0 ? 0 : pair);
      jf_linear_bwd(q, s, q + far, s + far, q + 2 * far, s + 2 * far, N, C, D, b, q + 3 * far, s + 3 * far, nullptr, q + 4 * far, s + 4 * far, nullptr, nullptr, 0, nullptr);
      if (seen.pairs != 1) { ++unforeseen; continue; }
      ++launched;
      const int td = (int)sd.tiles(d), tw = (int)sw.tiles(w), per = (td + tw + 255) / 256, resident = std::min(sd.resident, sw.resident);
      const double ud = sd.tile_us(kDgrad, d, per), uw = sw.tile_us(kWgrad, w, per);
      const int first = seen.second_first ? tw : td, second = seen.second_first ? td : tw;
      const PairDeal deal = {seen.deal[0], seen.deal[1], seen.deal[2], seen.deal[3]}, plain = {(first + 7) & ~7, 0, 0, 0};
      std::vector<double> load(256), in_order(256);
      for (int k = 0; k < seen.grid; ++k) {
        int tile = 0;
        bool early = deal.place(k, tile);
        if (tile < (early ? first : second)) load[k % 256] += early != (seen.second_first != 0) ? ud : uw;
        early = plain.place(k, tile);
        if (tile < (early ? first : second)) in_order[k % 256] += early != (seen.second_first != 0) ? ud : uw;
      }
      const double busiest = *std::max_element(load.begin(), load.end()), before = *std::max_element(in_order.begin(), in_order.end());
      worse += busiest > before + 1e-9;
      dealt += deal.few > 0;
      if (per > 1 && td + tw <= 256 * resident)
        unforeseen += p.fixed_us + p.work * (p.dealt * busiest + (1.0 - p.dealt) * (td * ud + tw * uw) / 256.0) > t.pair_us(p, d, w) + 1e-9;
    }
  }
  std::printf("launched %ld dealt %ld worse %ld unforeseen %ld\n", launched, dealt, worse, unforeseen);
  return worse || unforeseen || dealt < 500;
}
"""


def _run(tmp_path, source):
    src, exe = tmp_path / "deal.hip", tmp_path / "deal"
    src.write_text(source)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", CSRC, "-I", INCLUDE, str(src),
                    "-o", str(exe)], check=True, timeout=240)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout + res.stderr


def test_every_tile_once(tmp_path):
    _run(tmp_path, DEAL)


def test_the_deal_that_is_launched(tmp_path):
    """No compute unit has more to do than in order, by the times that the choice goes by, nor more than the choice counts on."""
    _run(tmp_path, LAUNCHED)


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
