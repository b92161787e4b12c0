// Which kernel a product runs on: tile shapes, pairs of products in one launch, and the rule that picks them.
//
// At B = 32 the products are bound by the vector ALU work of the per-K-block dequantization, which is the same per output
// element for every shape; what differs is what a wave pays per MFMA for fragment reads and staging (less for the larger
// wave tiles), how evenly the tiles fill 256 compute units, and the fixed cost of a tile.  The shapes, numbered as in
// jf_debug_set_gemm_shape:
//   1   128x128: four waves of 2x2 sub-blocks (B = 128: eight of 2x1), three workgroups per compute unit (B = 128: one)
//   4   64x64: four waves of one sub-block (not at B = 128)
//   6   256x128: eight waves of 2x2 sub-blocks; two workgroups per compute unit at B = 32, one at B = 128 (not at B = 64).
//       A quarter less operand traffic per MFMA than 128x128, and at B = 32 four waves per SIMD instead of three:
//       8192^3 991 -> 964 us
//   7   64x64 with a stage of 128 instead of 64 K bytes: half the barriers, three workgroups per compute unit (B = 32)
//   8   128x64: four waves of 2x1 sub-blocks, four workgroups per compute unit (B = 32)
//   10  32x32: four waves of 16x16 outputs, jf_gemm_fine.hpp (B = 32)
// A model of the busiest SIMD predicts the time of each and the least is taken.  Its constants are least-squares fits to the
// measured times of 276 products (92 layers drawn over the logarithm of their sizes, 128 .. 16384 tokens, 128 .. 8192
// features; all three products) and 184 backward passes: rms error 4-8 % for one shape (22 % for shape 10), and the shape
// taken is on average within 1.5 % (B = 32), 0.4 % (64) and 0.1 % (128) of the best one in each case; for the choice
// between one and two launches of the backward products within 1.7 %, 0.3 % and 0.2 %.
#pragma once
#include <algorithm>
#include <cmath>

#include "jf_gemm_kernel.hpp"

namespace jf {

// A workgroup puts `sub` 32x32 sub-blocks on every SIMD of its compute unit; with T tiles the busiest unit holds
// ceil(T / 256) workgroups while all are resident at once, T / 256 + tail beyond that.  A sub-block costs `ns` per 32 K on
// a SIMD shared by several workgroups, `ns_alone` on one that holds a single one (which cannot overlap its own MFMA, fold
// and waits), and `epilogue_us` besides; fixed_us is the launch and the latency of the first stage.
struct ShapeModel {
  int shape, tm, tn, resident;
  double sub, fixed_us, ns, ns_alone, tail, epilogue_us;

  double tiles(const GemmArgs& a) const { return (double)((a.M + tm - 1) / tm) * ((a.Nn + tn - 1) / tn); }
  double tile_us(const GemmArgs& a, double rate) const { return sub * (a.K / 32 * rate * 1e-3 + epilogue_us); }
  double product_us(const GemmArgs& a) const {
    const double t = tiles(a), busiest = t <= 256.0 * resident ? std::ceil(t / 256.0) : t / 256.0 + tail;
    return fixed_us + busiest * tile_us(a, busiest <= 1.0 ? ns_alone : ns);
  }
};

static constexpr ShapeModel kShapes32[] = {
    {6, 256, 128, 2, 8, 2.53, 53.6, 62.1, 0.73, 0.537}, {1, 128, 128, 3, 4, 3.69, 59.8, 88.3, 0.67, 0.478},
    {8, 128, 64, 4, 2, 3.51, 68.3, 105.9, 0.67, 0.490}, {4, 64, 64, 4, 1, 3.46, 82.9, 121.3, 1.20, 0.429},
    {7, 64, 64, 3, 1, 3.36, 76.9, 102.8, 0.92, 0.802},  {10, 32, 32, 4, 0.25, 3.84, 174.5, 223.5, 1.10, 1.263}};
static constexpr ShapeModel kShapes64[] = {{1, 128, 128, 3, 4, 3.36, 43.5, 61.9, 0.54, 0.421},
                                           {4, 64, 64, 3, 1, 3.29, 64.5, 75.6, 0.64, 0.769}};
static constexpr ShapeModel kShapes128[] = {{6, 256, 128, 1, 8, -0.19, 33.2, 28.5, 0.38, 0.860},
                                            {1, 128, 128, 1, 4, 2.23, 38.7, 33.6, 0.68, 0.808}};

// Both backward products in one launch: input gradient on shape `dgrad`, weight gradient on shape `wgrad`.  The compute
// units share the work of both, W = their average (more by 0.6 of what the rounding to whole workgroups adds while all are
// resident), so that the time is fixed_us + work * W + longest * (the longer tile's own time), at least that tile's time
// alone; with at most one tile per compute unit it is that.
struct PairModel {
  int pair, dgrad, wgrad;   // `pair` as in jf_debug_set_gemm_shape
  double fixed_us, work, longest;
};
static constexpr PairModel kPairs32[] = {{21, 1, 1, 3.56, 0.961, 0.191},  {22, 8, 8, 3.69, 1.002, 0.136},
                                         {23, 4, 4, 3.75, 1.127, -0.062}, {24, 10, 4, 3.98, 0.982, 0.416},
                                         {25, 4, 10, 3.98, 1.306, 0.167}};
static constexpr PairModel kPairs64[] = {{21, 1, 1, 3.36, 1.026, 0.097}, {22, 4, 4, 4.11, 0.986, 0.450}};
static constexpr PairModel kPairs128[] = {{21, 6, 6, -0.26, 1.013, 0.372}, {22, 1, 1, 2.23, 1.090, 0.107}};

struct ShapeTable {
  const ShapeModel* shapes;
  const PairModel* pairs;
  int nshapes, npairs;
  const ShapeModel* find(int shape) const {
    for (int i = 0; i < nshapes; ++i)
      if (shapes[i].shape == shape) return shapes + i;
    return nullptr;
  }
  const ShapeModel& best(const GemmArgs& a) const {
    const ShapeModel* b = shapes;
    for (int i = 1; i < nshapes; ++i)
      if (shapes[i].product_us(a) < b->product_us(a)) b = shapes + i;
    return *b;
  }
  double pair_us(const PairModel& p, const GemmArgs& d, const GemmArgs& w) const {
    const ShapeModel &sd = *find(p.dgrad), &sw = *find(p.wgrad);
    const double td = sd.tiles(d), tw = sw.tiles(w), per_cu = (td + tw) / 256.0;
    const double alone = std::max(sd.tile_us(d, sd.ns_alone), sw.tile_us(w, sw.ns_alone));
    if (per_cu <= 1.0) return p.fixed_us + alone;
    double work = (td * sd.tile_us(d, sd.ns) + tw * sw.tile_us(w, sw.ns)) / 256.0;
    if (per_cu <= std::min(sd.resident, sw.resident)) work *= 1.0 + 0.6 * (std::ceil(per_cu) / per_cu - 1.0);
    return p.fixed_us + std::max(alone, p.work * work + p.longest * alone);
  }
};
template <int NS, int NP>
static constexpr ShapeTable shape_table(const ShapeModel (&s)[NS], const PairModel (&p)[NP]) { return {s, p, NS, NP}; }
static inline ShapeTable shape_table(int block) {
  return block == 32 ? shape_table(kShapes32, kPairs32) : block == 64 ? shape_table(kShapes64, kPairs64) : shape_table(kShapes128, kPairs128);
}

// Shape of one product; `forced` (test hook) if that is a shape of this block size.
static int choose_shape(int block, const GemmArgs& a, int forced) {
  const ShapeTable t = shape_table(block);
  return t.find(forced) ? forced : t.best(a).shape;
}
// Pair of the backward products, 0 for two launches.
static int choose_pair(int block, const GemmArgs& dgrad, const GemmArgs& wgrad, int forced) {
  const ShapeTable t = shape_table(block);
  double least = t.best(dgrad).product_us(dgrad) + t.best(wgrad).product_us(wgrad);
  int pair = 0;
  for (int i = 0; i < t.npairs; ++i) {
    if (t.pairs[i].pair == forced) return forced;
    const double us = t.pair_us(t.pairs[i], dgrad, wgrad);
    if (us < least) least = us, pair = t.pairs[i].pair;
  }
  return forced ? 0 : pair;   // a forced shape means the single-product kernels
}

}  // namespace jf
