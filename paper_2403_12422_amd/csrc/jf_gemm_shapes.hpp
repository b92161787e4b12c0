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
//       8192^3 alone, forward / dgrad / wgrad: 990 / 965 / 951 us on 128x128, 943 / 940 / 933 us on 256x128
//   8   128x64: four waves of 2x1 sub-blocks, four workgroups per compute unit (B = 32)
//   10  32x32: four waves of 16x16 outputs, jf_gemm_fine.hpp (B = 32)
//   11  256x256: eight waves of 2x4 sub-blocks in persistent workgroups, one per compute unit, jf_gemm_wide.hpp (B = 64, 128)
// A model of the busiest SIMD predicts the time of each and the least is taken.  Its constants are least-squares fits to the
// measured times of 276 products (92 layers drawn over the logarithm of their sizes, 128 .. 16384 tokens, 128 .. 8192
// features; all three products) and 184 backward passes: rms error 4-9 % for one shape, and the shape taken is on
// average within 0.8 % (B = 32) of the best one in each case; for the choice between one and two launches of the backward
// products within 1.3 %.  With shape 11, whose constants and those of the pairs at B = 128 are fitted to 540 products and 180
// backward passes per block size: 0.5 % (B = 64) and 0.2 % (128), pairs 0.2 % and 0.8 %.  Over the same layers shape 11 is taken
// for 11 % (B = 64) and 44 % (128) of the products and gains 0.9 % and 7.0 % on the average of all.
#pragma once
#include <algorithm>
#include <cmath>

#include "jf_gemm_kernel.hpp"

namespace jf {

// A workgroup puts `sub` 32x32 sub-blocks on every SIMD of its compute unit; with T tiles the busiest unit holds
// ceil(T / 256) workgroups while all are resident at once, T / 256 + tail beyond that.  A sub-block costs `ns` per 32 K on
// a SIMD shared by several workgroups, `ns_alone` on one that holds a single one (which cannot overlap its own MFMA, fold
// and waits) in the forward product, `dgrad` and `wgrad` times that in the others, whose operands are read transposed, and
// `epilogue_us` besides; fixed_us is the launch and the latency of the first stage.
static constexpr int kPersistent = 1 << 24;   // as many as the largest output has
enum Product { kForward, kDgrad, kWgrad };
struct ShapeModel {
  int shape, tm, tn, resident;
  double sub, fixed_us, ns, ns_alone, tail, epilogue_us, dgrad, wgrad;

  double tiles(const GemmArgs& a) const { return (double)((a.M + tm - 1) / tm) * ((a.Nn + tn - 1) / tn); }
  double tile_us(Product p, const GemmArgs& a, bool alone) const {
    const double rate = (alone ? ns_alone : ns) * (p == kForward ? 1.0 : p == kDgrad ? dgrad : wgrad);
    return sub * (a.K / 32 * rate * 1e-3 + epilogue_us);
  }
  double product_us(Product p, const GemmArgs& a) const {
    // (a persistent workgroup takes whole tiles by turns, however many there are: `resident` is kPersistent there)
    const double t = tiles(a), busiest = t <= 256.0 * resident ? std::ceil(t / 256.0) : t / 256.0 + tail;
    return fixed_us + busiest * tile_us(p, a, busiest <= 1.0);
  }
};

static constexpr ShapeModel kShapes32[] = {
    {6, 256, 128, 2, 8, 2.25, 51.8, 60.0, 0.78, 0.524, 1.028, 1.039},
    {1, 128, 128, 3, 4, 3.11, 58.8, 87.2, 0.68, 0.480, 1.021, 0.995},
    {8, 128, 64, 4, 2, 2.98, 66.8, 103.3, 0.65, 0.501, 1.026, 1.020},
    {4, 64, 64, 4, 1, 2.95, 68.5, 109.1, 1.03, 0.703, 1.074, 1.206},
    {10, 32, 32, 4, 0.25, 3.26, 110.0, 125.5, 0.72, 1.798, 1.511, 2.205}};
static constexpr ShapeModel kShapes64[] = {
    {1, 128, 128, 3, 4, 2.82, 42.2, 58.5, 0.51, 0.464, 0.967, 1.001},
    {4, 64, 64, 3, 1, 2.71, 58.3, 66.0, 0.59, 0.827, 1.055, 1.237},
    {11, 256, 256, kPersistent, 16, 0.0, 41.3, 38.4, 0.0, 0.490, 0.995, 0.990}};
static constexpr ShapeModel kShapes128[] = {
    {6, 256, 128, 1, 8, -1.22, 29.8, 25.3, 0.38, 0.945, 1.014, 1.070},
    {1, 128, 128, 1, 4, 1.44, 34.2, 30.7, 0.79, 0.890, 1.001, 1.046},
    {11, 256, 256, kPersistent, 16, 0.0, 25.1, 21.8, 0.0, 0.474, 0.993, 1.015}};

// Both backward products in one launch: input gradient on shape `dgrad`, weight gradient on shape `wgrad`.  The compute
// units share the work of both, W = their average (more by 0.6 of what the rounding to whole workgroups adds while all are
// resident), so that the time is fixed_us + work * W + longest * (the longer tile's own time), at least that tile's time
// alone; with at most one tile per compute unit it is that.
struct PairModel {
  int pair, dgrad, wgrad;   // `pair` as in jf_debug_set_gemm_shape
  double fixed_us, work, longest;
};
static constexpr PairModel kPairs32[] = {{21, 1, 1, 3.14, 0.922, 0.243}, {22, 8, 8, 3.15, 0.986, 0.148}, {23, 4, 4, 2.69, 0.998, 0.310},
                                         {24, 10, 4, 2.91, 0.974, 0.378}, {25, 4, 10, 2.64, 1.032, 0.217}};
// Pair 26 is one list of tiles dealt to persistent workgroups: time = work * (the longest workgroup's tiles).
static constexpr PairModel kPairs64[] = {{21, 1, 1, 2.71, 0.983, 0.204}, {22, 4, 4, 2.93, 0.945, 0.385}, {26, 11, 11, 0.0, 0.973, 0.0}};
static constexpr PairModel kPairs128[] = {{21, 6, 6, -1.50, 0.910, 0.310}, {22, 1, 1, 1.46, 1.090, 0.118}, {26, 11, 11, 0.0, 1.011, 0.0}};

struct ShapeTable {
  const ShapeModel* shapes;
  const PairModel* pairs;
  int nshapes, npairs;
  const ShapeModel* find(int shape) const {
    for (int i = 0; i < nshapes; ++i)
      if (shapes[i].shape == shape) return shapes + i;
    return nullptr;
  }
  struct Choice {
    int shape;
    double us;
  };
  Choice best(Product p, const GemmArgs& a) const {
    Choice c = {shapes[0].shape, shapes[0].product_us(p, a)};
    for (int i = 1; i < nshapes; ++i) {
      const double us = shapes[i].product_us(p, a);
      if (us < c.us) c = {shapes[i].shape, us};
    }
    return c;
  }
  double pair_us(const PairModel& p, const GemmArgs& d, const GemmArgs& w) const {
    const ShapeModel &sd = *find(p.dgrad), &sw = *find(p.wgrad);
    if (sd.resident == kPersistent) {
      // as gemm_wide_pair_kernel deals them; the workgroup with most tiles is the first of either product
      const bool second_first = w.K > d.K;
      const int64_t td = (int64_t)sd.tiles(d), tw = (int64_t)sw.tiles(w), t1 = second_first ? tw : td, t2 = second_first ? td : tw;
      const double us_d = sd.tile_us(kDgrad, d, false), us_w = sw.tile_us(kWgrad, w, false);
      const int64_t split = (t1 + 7) & ~int64_t(7), n = std::min<int64_t>(256, split + t2);
      double busiest = 0.0;
      for (const int64_t i : {int64_t(0), split % n}) {
        const int64_t n1 = i < t1 ? (t1 - i + n - 1) / n : 0, j = (n - split % n + i) % n, n2 = j < t2 ? (t2 - j + n - 1) / n : 0;
        busiest = std::max(busiest, n1 * (second_first ? us_w : us_d) + n2 * (second_first ? us_d : us_w));
      }
      return p.fixed_us + p.work * busiest;
    }
    const double td = sd.tiles(d), tw = sw.tiles(w), per_cu = (td + tw) / 256.0;
    const double alone = std::max(sd.tile_us(kDgrad, d, true), sw.tile_us(kWgrad, w, true));
    if (per_cu <= 1.0) return p.fixed_us + alone;
    double work = (td * sd.tile_us(kDgrad, d, false) + tw * sw.tile_us(kWgrad, w, false)) / 256.0;
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
static int choose_shape(int block, Product p, const GemmArgs& a, int forced) {
  const ShapeTable t = shape_table(block);
  return t.find(forced) ? forced : t.best(p, a).shape;
}
// Pair of the backward products, 0 for two launches.
static int choose_pair(int block, const GemmArgs& dgrad, const GemmArgs& wgrad, int forced) {
  const ShapeTable t = shape_table(block);
  double least = t.best(kDgrad, dgrad).us + t.best(kWgrad, wgrad).us;
  int pair = 0;
  for (int i = 0; i < t.npairs; ++i) {
    if (t.pairs[i].pair == forced) return forced;
    const double us = t.pair_us(t.pairs[i], dgrad, wgrad);
    if (us < least) least = us, pair = t.pairs[i].pair;
  }
  return forced ? 0 : pair;   // a forced shape means the single-product kernels
}

}  // namespace jf
