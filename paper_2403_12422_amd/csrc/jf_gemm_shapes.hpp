// Which kernel a product runs on: tile shapes, pairs of products in one launch, and the rule that picks them.
//
// At B = 32 the products are bound by the vector ALU work of the per-K-block dequantization, which is the same per output
// element for every shape; what differs is what a wave pays per MFMA for fragment reads and staging (less for the larger
// wave tiles), how evenly the tiles fill 256 compute units, and the fixed cost of a tile.  The shapes, numbered as in
// jf_debug_set_gemm_shape:
//   1   128x128: four waves of 2x2 sub-blocks (B = 128: eight of 2x1), three workgroups per compute unit (B = 128: one)
//   4   64x64: four waves of one sub-block (not at B = 128)
//   6   256x128: eight waves of 2x2 sub-blocks; two workgroups per compute unit at B = 32, one at B = 128 (not at B = 64).
//       A quarter less operand traffic per MFMA than 128x128, and at B = 32 four waves per SIMD instead of three (8192^3 969 -> 939 us)
//   7   128x64: eight waves of one sub-block, three workgroups per compute unit (B = 32).  More fragment reads per MFMA than 8, but
//       twice the waves: up to six on a SIMD, where one or two tiles a unit leave 8 a wave or two (2048^3 alone 21.6 -> 20.0 us); 8 keeps
//       outputs of little K in three to four tiles a unit (4704 x 992 x 320 8.6 and 10.2)
//   8   128x64: four waves of 2x1 sub-blocks, four workgroups per compute unit (B = 32)
//   10  32x32: four waves of 16x16 outputs, jf_gemm_fine.hpp (B = 32)
//   11  256x256: eight waves of 2x4 sub-blocks in persistent workgroups, one per compute unit, jf_gemm_wide.hpp (B = 64, 128)
// (More in profiles/kernel_choice.txt.)
// A model of the busiest compute unit predicts the time of each and the least is taken.  Its constants are least-squares fits to the
// measured times of all shapes and pairs on 400 (B = 32) and 280 (64, 128) layers, half of them drawn over the logarithm of their
// sizes (128 .. 16384 tokens, 128 .. 11008 features), half from multiples of 256: rms error 3-8 % for one shape.  Fitted to every other
// layer, the choice costs on the rest, against the best shape or pair of each, on average 0.3 % (B = 64) and 0.0 % (128) for single
// products and 0.2 and 0.5 % for backward passes (their forerunner, without rounds, resident counts and distant operands, 0.7 and 1.9).
// At B = 32 shape 7 and pair 26 were fitted with the rest held, every layer scaled by the shapes that both fits know; on 120 further
// layers the choice costs 0.6 % for single products (without shape 7 1.2).  Backward passes on the kernels and deals as they are now, 820 other
// layers at B = 32 and 100 each at 64 and 128, by replays of graphs: 1.0, 0.5 and 0.7 %, of which the measurement's own noise
// is up to 0.5 (the pairs' constants fitted anew to half of 560 of these layers: 1.2 to 1.4 % on the other half, so they stay).  At B = 32 one layer in nine loses more than 3 %, nearly half of them beyond one residency, where a pair counts with the mean time of its
// tiles though the last long ones end it alone: 2048 x 768 -> 7168 61 us on pair 23, 48 on 26; 9216 x 2560 -> 1024 114 and 105.
// At B = 128 with both products on shape 11 one launch and two are within 2 % of each other: 4096^3 138.8 and 141.4 us, 8192 x 4096 -> 4096 265.7
// and 268.0, 16384 x 4096 -> 11008 1428 and 1412.
// (Shape 11 has been scaled by what it has gained since: at B = 128 4.3 % forward, 5.7 % input gradient, 1.5 % weight gradient, at B = 64 1.6, 3.3 and
// 3.4 %.)
#pragma once
#include <algorithm>
#include <cmath>

#include "jf_gemm_kernel.hpp"

namespace jf {

// A workgroup puts `sub` 32x32 sub-blocks on every SIMD of its compute unit.  A sub-block costs ns[n - 1] per 32 K with n workgroups
// resident (one alone cannot overlap its own MFMA, fold and waits) in the forward product, `dgrad` and `wgrad` times that in the
// others, whose operands are read transposed, up to 1 + `far` times that where the operands are too large for the caches, and
// `epilogue_us` besides; fixed_us is the launch and the latency of the first stage.
static constexpr int kPersistent = 1 << 24;   // as many as the largest output has
enum Product { kForward, kDgrad, kWgrad };
struct ShapeModel {
  int shape, tm, tn, resident;
  double sub, fixed_us, tail, epilogue_us, dgrad, wgrad, far, fade, ns[4];

  double tiles(const GemmArgs& a) const { return (double)((a.M + tm - 1) / tm) * ((a.Nn + tn - 1) / tn); }
  // one tile's share of its unit with n workgroups resident
  double tile_us(Product p, const GemmArgs& a, int n) const {
    const double mb = ((double)a.M + a.Nn) * a.K * 1e-6, rate = ns[std::min(n, 4) - 1] * (1.0 + far * mb / (mb + 20.0));
    return sub * (a.K / 32 * rate * (p == kForward ? 1.0 : p == kDgrad ? dgrad : wgrad) * 1e-3 + epilogue_us);
  }
  double product_us(Product p, const GemmArgs& a) const;
};

// Time of `per` workgroups a compute unit, u(n) each with n resident: whole rounds of `resident`, then the rest by itself, fewer
// workgroups to a unit.  The more rounds have gone before, the less do workgroups end together (`fade` a round): then the rest runs
// beside the others, and `tail` is what the last ones add.
// (A persistent workgroup takes whole tiles by turns, however many there are: `resident` is kPersistent there.)
template <class U>
static double rounds_us(double per, int resident, const U& u, double fade, double tail) {
  if (per <= resident) {
    const int n = (int)std::ceil(per);
    return n * u(n);
  }
  const double k = std::floor(per / resident), rest = per - k * resident, together = std::pow(fade, k);
  const int n = (int)std::ceil(rest);
  return k * resident * u(resident) + (n ? together * n * u(n) : 0.0) + (1.0 - together) * (rest + tail) * u(resident);
}
inline double ShapeModel::product_us(Product p, const GemmArgs& a) const {
  return fixed_us + rounds_us(tiles(a) / 256.0, resident, [&](int n) { return tile_us(p, a, n); }, fade, tail);
}

static constexpr ShapeModel kShapes32[] = {
    {6, 256, 128, 2, 8, 2.788, 2.368, 0.4550, 1.021, 1.031, 0.0952, 0.923, {56.07, 45.61, 45.61, 45.61}},
    {1, 128, 128, 3, 4, 3.457, 1.268, 0.3633, 1.020, 0.994, 0.0545, 0.837, {82.35, 53.42, 51.33, 51.33}},
    {7, 128, 64, 3, 2, 2.653, 1.035, 0.6787, 1.019, 1.025, 0.2504, 0.904, {67.30, 48.65, 47.49, 47.49}},
    {8, 128, 64, 4, 2, 2.956, 1.145, 0.4533, 1.016, 0.999, 0.1229, 0.788, {96.07, 60.13, 55.10, 56.05}},
    {4, 64, 64, 4, 1, 2.801, 2.493, 0.7624, 1.061, 1.182, 0.3667, 0.990, {97.87, 56.00, 50.30, 50.06}},
    {10, 32, 32, 4, 0.25, 3.209, 1.020, 2.0237, 1.654, 2.570, 0.5469, 1.000, {105.91, 80.90, 81.07, 70.29}}};
static constexpr ShapeModel kShapes64[] = {
    {1, 128, 128, 3, 4, 3.314, 3.011, 0.3236, 1.005, 1.015, 0.0838, 0.905, {53.31, 36.74, 36.44, 36.44}},
    {4, 64, 64, 3, 1, 2.834, 4.580, 0.8016, 1.177, 1.387, 0.2486, 0.948, {54.10, 41.61, 40.66, 40.66}},
    {11, 256, 256, kPersistent, 16, 2.233, 0.0, 0.3669, 1.000, 1.021, 0.1604, 0.0, {30.88, 34.13, 34.13, 34.13}}};
static constexpr ShapeModel kShapes128[] = {
    {6, 256, 128, 1, 8, 1.976, 4.369, 0.5626, 0.997, 1.017, 0.1561, 0.933, {23.17, 23.17, 23.17, 23.17}},
    {1, 128, 128, 1, 4, 1.701, 13.765, 0.7992, 1.011, 1.080, 0.1634, 0.986, {27.13, 27.13, 27.13, 27.13}},
    {11, 256, 256, kPersistent, 16, 2.794, 0.0, 0.3786, 1.015, 1.031, 0.2910, 0.0, {18.07, 20.98, 20.98, 20.98}}};

// Both backward products in one launch: input gradient on shape `dgrad`, weight gradient on shape `wgrad`, the longer tiles dealt
// first.  While all are resident the busiest unit counts for `dealt` and the average for the rest; beyond that whole rounds and a rest
// as above, of tiles of the mean time.  `work` is what running side by side saves or costs; never less than one tile alone.
struct PairModel {
  int pair, dgrad, wgrad;   // `pair` as in jf_debug_set_gemm_shape
  double fixed_us, work, dealt, fade;
};
static constexpr PairModel kPairs32[] = {{21, 1, 1, 3.749, 1.062, 0.671, 0.556}, {22, 8, 8, 3.269, 1.040, 0.795, 0.653},
                                         {23, 4, 4, 3.093, 1.017, 0.974, 1.0},   {24, 10, 4, 3.230, 1.004, 1.153, 1.0},
                                         {25, 4, 10, 3.314, 1.013, 0.808, 1.0},   {26, 7, 7, 3.041, 1.050, 0.844, 0.801}};
static constexpr PairModel kPairs64[] = {{21, 1, 1, 3.762, 1.062, 0.708, 0.665}, {22, 4, 4, 3.225, 1.088, 0.669, 0.747},
                                         {26, 11, 11, 2.822, 1.037, 0.825, 0.0}};
static constexpr PairModel kPairs128[] = {{21, 6, 6, 2.371, 1.284, 0.800, 0.416}, {22, 1, 1, 2.089, 1.212, 0.800, 0.596},
                                          {26, 11, 11, 4.458, 1.089, 0.737, 0.0}};

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
  // Time of a pair and, in *order, how its tiles are dealt: the product with the larger K times tile first, by turns or as deal_pair
  // says.
  double pair_us(const PairModel& p, const GemmArgs& d, const GemmArgs& w, PairChoice* order = nullptr) const {
    const ShapeModel &sd = *find(p.dgrad), &sw = *find(p.wgrad);
    const auto ud = [&](int n) { return sd.tile_us(kDgrad, d, n); };
    const auto uw = [&](int n) { return sw.tile_us(kWgrad, w, n); };
    const double td = sd.tiles(d), tw = sw.tiles(w), per = (td + tw) / 256.0, alone = std::max(ud(1), uw(1));
    const int resident = std::min(sd.resident, sw.resident);
    const bool second_first = (int64_t)w.K * sw.tm * sw.tn > (int64_t)d.K * sd.tm * sd.tn;
    const int t1 = (int)(second_first ? tw : td), t2 = (int)(second_first ? td : tw);
    PairChoice in_order = {p.pair, second_first, {(t1 + 7) & ~7, 0, 0, 0}};
    PairChoice& o = order ? *order : in_order;
    o = in_order;
    if (per <= 1.0) return p.fixed_us + alone;
    if (per > resident) {
      const auto mean = [&](int n) { return (td * ud(n) + tw * uw(n)) / (td + tw); };
      return p.fixed_us + std::max(alone, p.work * rounds_us(per, resident, mean, p.fade, 0.0));
    }
    const int n = (int)std::ceil(per);
    const double u1 = second_first ? uw(n) : ud(n), u2 = second_first ? ud(n) : uw(n);
    double busiest = 0.0;
    o.deal = deal_pair(t1, t2, u1, u2, sd.resident == kPersistent ? 0 : resident, &busiest);   // (persistent workgroups: in order)
    const double average = (t1 * u1 + t2 * u2) / 256.0;
    return p.fixed_us + std::max(alone, p.work * (p.dealt * busiest + (1.0 - p.dealt) * average));
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
// Pair of the backward products and the order of its tiles.
static PairChoice choose_pair(int block, const GemmArgs& dgrad, const GemmArgs& wgrad, int forced) {
  const ShapeTable t = shape_table(block);
  double least = t.best(kDgrad, dgrad).us + t.best(kWgrad, wgrad).us;
  PairChoice c = {};
  for (int i = 0; i < t.npairs; ++i) {
    PairChoice order;
    const double us = t.pair_us(t.pairs[i], dgrad, wgrad, &order);
    if (t.pairs[i].pair == forced) return order;
    if (us < least) least = us, c = order;
  }
  return forced ? PairChoice{} : c;   // a forced shape means the single-product kernels
}

}  // namespace jf
