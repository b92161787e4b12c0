// LayerNorm of few row groups at block size 32: one pass as in jf_layernorm_rows.hpp, each row group shared by several workgroups.
//
// What bounds these tensors is one wave's chain of 64 elements per lane, with most compute units idle beside it (1056 x 800 has
// 33 row groups for 256 units).  The sums of a row are the cheap part of it -- two integer dot products for four codes forward,
// five instructions an element backward -- so PARTS workgroups form them from the whole rows, each for itself, and
// each goes on with its part of every strip: one block of the four, or two.  The sums are those of the one-pass kernels, in the
// same order, and so are the results.
// Forward / backward in us: 128 x 128 4.1 -> 3.55 / 4.45 -> 4.2, 1056 x 800 5.4 -> 4.75 / 6.6 -> 5.9, 1024 x 2048 7.9 -> 6.65 / 11.0 -> 9.05,
// 2048 x 768 5.4 -> 4.75 / 7.9 -> 6.85, 4096 x 768 5.6 -> 4.95 / 9.4 -> 8.4.  What is left is mostly the launch, the way to memory and back
// (an empty kernel 1.6, 1 MB copied 1.7), and the rows themselves, of which a compute unit gets 26 bytes a nanosecond.
#include "jf_layernorm_rows.hpp"

namespace jf {

// Part `part` of row group `group`: the parts of a group are 8 workgroups apart, on one XCD, whose L2 then fetches the rows once.
struct SplitPlace {
  int group, part;
  template <int PARTS>
  static __device__ __forceinline__ SplitPlace of(unsigned index) {
    SplitPlace s;
    s.part = (int)(index / 8 % PARTS);
    s.group = (int)(index / (8 * PARTS) * 8 + index % 8);
    return s;
  }
};
template <int PARTS>
static int split_grid(int groups) { return (groups + 7) / 8 * 8 * PARTS; }

// Second lane mapping of a wave, for its part of the strip: pass p has chunk `chunk` of row row0 + PASS_ROWS p.  The lanes of a
// block are the whole wave (four parts) or half of it.
template <int PARTS>
struct SplitLane {
  static_assert(PARTS == 2 || PARTS == 4, "one or two of a strip's four blocks");
  static constexpr int PASSES = 4 / PARTS, PASS_ROWS = 32 / PASSES, BLOCK_LANES = PARTS == 4 ? 63 : 31;
  int chunk, row0;
  __device__ __forceinline__ SplitLane(int part, int lane) {
    chunk = part * (8 / PARTS) + (lane & 1) + (PARTS == 2 ? 2 * (lane >> 5) : 0);
    row0 = (lane >> 1) & (PASS_ROWS - 1);
  }
};

// Eq. 1 on a wave's part and its stores
template <int PARTS>
__device__ __forceinline__ void store_part_of_strip(const float (&y)[SplitLane<PARTS>::PASSES][16], const SplitLane<PARTS>& s, int lane, bool ok, int col,
                                                    int64_t first_row, int cols, int8_t* Y, float* SY) {
  typedef SplitLane<PARTS> L;
  float m = 0.0f;
#pragma unroll
  for (int p = 0; p < L::PASSES; ++p) m = amax16(m, y[p]);
  m = wave_group_max<L::BLOCK_LANES>(m);
  float scale;
  double inv;
  block_scale(m, scale, inv);
  if (!ok) return;
#pragma unroll
  for (int p = 0; p < L::PASSES; ++p) store_out(Y + (first_row + s.row0 + L::PASS_ROWS * p) * cols + col, quantize16(y[p], inv));
  if ((lane & L::BLOCK_LANES) == 0) store_out(SY + first_row / 32 * (cols / 32) + col / 32, scale);
}

template <bool PARTIALS, int PARTS>
__global__ void __launch_bounds__(1024) layernorm_split_kernel(const int8_t* X, const float* SX, const float* first_in, const float* second_in, int rows,
                                                               int cols, int layout, int, const LayerNormRows) {
  extern __shared__ __align__(16) int8_t smem[];
  LayerNormRows a = first_arguments<PARTIALS>(X, SX, first_in, second_in, rows, cols, layout);
  const SplitPlace place = SplitPlace::of<PARTS>(blockIdx.x);
  const int g = place.group, lc = a.cols / 32;
  if (g >= a.rows / 32) return;
  const RowWave t(a.cols, layout);
  double* const s_row = reinterpret_cast<double*>(smem);
  int8_t* const own = smem + t.waves * kFwdRowBytes + t.wave * kFwdWaveBytes;
  const int8_t* const x = uniform_pointer(a.X + (int64_t)g * 32 * a.cols);
  const uint32_t off = (uint32_t)(t.rsub * a.cols + t.col);
#pragma unroll
  for (int p = 0; p < 4; ++p) load_lds_16(x + (int64_t)p * 8 * a.cols, off, own, 1024 * p);
  load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SX + (int64_t)g * lc)), (uint32_t)(t.col / 32) * 4, own, kFwdScale);
  if (PARTIALS) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t o = (int64_t)min(4 * t.strip + 2 * i + (t.lane >> 5), lc - 1) * a.rows + g * 32 + (t.lane & 31);
      load_lds_4_vaddr(a.row_mean + o, own, kFwdPart + 256 * i);
      load_lds_4_vaddr(a.row_sumsq + o, own, kFwdPart + 512 + 256 * i);
    }
  }
  other_arguments<PARTIALS>(a);
  const SplitLane<PARTS> s(place.part, t.lane);
  const bool ok = t.c0 + 16 * s.chunk < a.cols;
  const int col = ok ? t.c0 + 16 * s.chunk : t.c0;
  float gm[16], bt[16];
  load16f(a.gamma + col, gm);
  load16f(a.beta + col, bt);
  wait_all_loads();
  wave_lds_fence();

  // the sums of the rows, as in layernorm_rows_kernel
  double* const row = s_row + t.wave * 32 * 2;
  if (PARTIALS) {
    const float* part = reinterpret_cast<const float*>(own + kFwdPart) + 128 * (t.lane >> 5) + (t.lane & 31);
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) v += 4 * t.strip + j < lc ? (double)part[32 * j] : 0.0;
    row[2 * (t.lane & 31) + (t.lane >> 5)] = v;
  } else {
    const double sd = t.ok ? (double)*reinterpret_cast<const float*>(own + kFwdScale + 4 * t.lane) : 0.0, sd2 = sd * sd;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      int s1, s2;
      chunk_moments(*reinterpret_cast<const uint4*>(own + 1024 * p + 16 * t.lane), s1, s2);
      s1 += lane_xor_i32<0>(s1);
      s2 += lane_xor_i32<0>(s2);
      double m1 = sd * (double)s1, m2 = sd2 * (double)s2;
      m1 += lane_xor_f64<1>(m1);
      m2 += lane_xor_f64<1>(m2);
      m1 += lane_xor_f64<2>(m1);
      m2 += lane_xor_f64<2>(m2);
      if (t.ch == 0) *reinterpret_cast<double2*>(row + 2 * (t.rsub + 8 * p)) = make_double2(m1, m2);
    }
  }
  lds_barrier();
  {
    const double sum = sum_over_strips(s_row + (t.lane & 31) * 2 + (t.lane >> 5), a.strips), other = lane_xor_f64<5>(sum);
    const double mud = (t.lane < 32 ? sum : other) * (PARTIALS ? a.inv_blocks : a.inv_cols);
    const float var = fmaxf((float)((t.lane < 32 ? other : sum) * a.inv_cols - mud * mud), 0.0f);
    const float ve = var + a.eps;
    float rs = __builtin_amdgcn_rsqf(ve);
    rs = rs * __builtin_fmaf(-0.5f * ve * rs, rs, 1.5f);
    if (t.lane < 32) reinterpret_cast<float2*>(own + kFwdStat)[t.lane] = make_float2((float)mud, rs);
    wave_lds_fence();
    if (place.part == 0 && t.strip == 0 && t.lane < 32) {
      a.mean[g * 32 + t.lane] = (float)mud;
      a.rstd[g * 32 + t.lane] = rs;
    }
  }
  const float sx = *reinterpret_cast<const float*>(own + kFwdScale + 4 * s.chunk);
  float y[s.PASSES][16];
#pragma unroll
  for (int p = 0; p < s.PASSES; ++p) {
    const int r = s.row0 + s.PASS_ROWS * p;
    const float2 st = reinterpret_cast<const float2*>(own + kFwdStat)[r];
    const float k1 = sx * st.y, kb = __builtin_fmaf(-128.0f, k1, -st.x * st.y);
    float u[16];
    unpack16_biased(*reinterpret_cast<const uint4*>(own + 128 * r + 16 * s.chunk), u);
#pragma unroll
    for (int e = 0; e < 16; ++e) y[p][e] = __builtin_fmaf(__builtin_fmaf(u[e], k1, kb), gm[e], bt[e]);
  }
  store_part_of_strip<PARTS>(y, s, t.lane, ok, col, (int64_t)g * 32, a.cols, a.Y, a.SY);
}

// Sums over the sixteen lanes that differ in bits 1 to 4 of 16 values, by halves as in reduce_rows_of_32 (lanes with the bit clear go on
// with one value of a pair, with it set with the other): 50 instructions.  A lane ends with value (lane / 2) % 16.
__device__ __forceinline__ float reduce_sixteen_rows(const float (&a)[16], int lane) {
  const auto bits = [](float x) __attribute__((always_inline)) { return __builtin_bit_cast(int, x); };
  const auto real = [](int x) __attribute__((always_inline)) { return __builtin_bit_cast(float, x); };
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const auto p = __builtin_amdgcn_permlane16_swap(bits(a[j]), bits(a[j + 8]), false, false);
    v[j] = real((int)p[0]) + real((int)p[1]);
  }
  constexpr int SAME = 0xE4;   // quad_perm [0,1,2,3]
#pragma unroll
  for (int j = 0; j < 4; ++j) {   // across 8 lanes
    const int mine = __builtin_amdgcn_update_dpp(bits(v[j]), bits(v[j + 4]), SAME, 0xf, 0xC, false);
    const int other = __builtin_amdgcn_update_dpp(bits(v[j + 4]), bits(v[j]), SAME, 0xf, 0xC, false);
    v[j] = real(mine) + real(__builtin_amdgcn_mov_dpp(other, 0x128, 0xf, 0xf, false));
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {   // across 4 lanes: row_shl and row_shr, each for the lanes that it is right for
    const int mine = __builtin_amdgcn_update_dpp(bits(v[j]), bits(v[j + 2]), SAME, 0xf, 0xA, false);
    const int other = __builtin_amdgcn_update_dpp(bits(v[j + 2]), bits(v[j]), SAME, 0xf, 0xA, false);
    const int low = __builtin_amdgcn_update_dpp(other, other, 0x104, 0xf, 0x5, false);
    v[j] = real(mine) + real(__builtin_amdgcn_update_dpp(low, other, 0x114, 0xf, 0xA, false));
  }
  const bool second = (lane & 2) != 0;   // across 2 lanes
  return (second ? v[1] : v[0]) + lane_xor_f32<1>(second ? v[0] : v[1]);
}

// Backward.  Column sums: in workgroups of their own behind row_wgs that have rows (column_sums_direct; waves past the strips are for
// those only), or, COLUMNS, each workgroup's of its part, as one partial row for a row group, which another launch adds: where the rows
// of many groups take a chip by themselves.
template <int PARTS, bool COLUMNS>
__global__ void __launch_bounds__(1024) layernorm_bwd_split_kernel(const int8_t* G, const float* SG, const int8_t* X, const float* SX, int rows, int cols,
                                                                   int layout, int wgs, const float* gamma, const LayerNormBwdRows) {
  extern __shared__ __align__(16) int8_t smem[];
  LayerNormBwdRows a = first_arguments(G, SG, X, SX, rows, cols, layout, wgs, gamma);
  if (!COLUMNS && (int)blockIdx.x >= a.row_wgs) {
    other_arguments(a);
    column_sums_direct<32>(a, blockIdx.x - a.row_wgs, layout >> 16, reinterpret_cast<float*>(smem));
    return;
  }
  const SplitPlace place = SplitPlace::of<PARTS>(blockIdx.x);
  const int g = place.group, lc = a.cols / 32;
  const RowWave t(a.cols, layout);
  if (g >= a.rows / 32 || t.team > 0) return;
  float* const s_row = reinterpret_cast<float*>(smem);
  int8_t* const own = smem + a.strips * kBwdRowBytes + t.wave * kBwdWaveBytes;
  const int8_t* const x = uniform_pointer(a.X + (int64_t)g * 32 * a.cols);
  const int8_t* const gr = uniform_pointer(a.G + (int64_t)g * 32 * a.cols);
  const uint32_t off = (uint32_t)(t.rsub * a.cols + t.col), off_scale = (uint32_t)(t.col / 32) * 4;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    load_lds_16(x + (int64_t)p * 8 * a.cols, off, own, 1024 * p);
    load_lds_16(gr + (int64_t)p * 8 * a.cols, off, own, kBwdG + 1024 * p);
  }
  load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SX + (int64_t)g * lc)), off_scale, own, kBwdScaleX);
  load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SG + (int64_t)g * lc)), off_scale, own, kBwdScaleG);
  other_arguments(a);
  if (t.lane < 32) {
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.mean + g * 32)), (uint32_t)t.lane * 4, own, kBwdMean);
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.rstd + g * 32)), (uint32_t)t.lane * 4, own, kBwdRstd);
  }
  float* const s_gamma = reinterpret_cast<float*>(own + kBwdGamma);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = t.c0 + t.lane + 64 * i;
    s_gamma[t.lane + 64 * i] = c < a.cols ? a.gamma[c] : 0.0f;
  }
  wait_all_loads();
  wave_lds_fence();

  // the two sums of each row, as in layernorm_bwd_rows_kernel
  float* const row = s_row + t.wave * 32 * 2;
  {
    const float sx = *reinterpret_cast<const float*>(own + kBwdScaleX + 4 * t.lane);
    const float sg = t.ok ? *reinterpret_cast<const float*>(own + kBwdScaleG + 4 * t.lane) : 0.0f;
    float kx[4], cx[4], m1[4], m2[4];
    uint4 px[4], pg[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      px[p] = *reinterpret_cast<const uint4*>(own + 1024 * p + 16 * t.lane);
      pg[p] = *reinterpret_cast<const uint4*>(own + kBwdG + 1024 * p + 16 * t.lane);
      const float rs = reinterpret_cast<const float*>(own + kBwdRstd)[t.rsub + 8 * p];
      kx[p] = sx * rs;
      cx[p] = -reinterpret_cast<const float*>(own + kBwdMean)[t.rsub + 8 * p] * rs;
      m1[p] = m2[p] = 0.0f;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const float4 gm4 = *reinterpret_cast<const float4*>(s_gamma + 16 * t.ch + 4 * d);
      const float gm[4] = {gm4.x, gm4.y, gm4.z, gm4.w};
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float xc[4], gc[4];
        unpack4(dword_of(px[p], d), xc);
        unpack4(dword_of(pg[p], d), gc);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gh = gc[e] * gm[e];
          m1[p] += gh;
          m2[p] = __builtin_fmaf(gh, __builtin_fmaf(xc[e], kx[p], cx[p]), m2[p]);
        }
      }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      m1[p] = wave_group_sum<7>(m1[p] * sg);
      m2[p] = wave_group_sum<7>(m2[p] * sg);
      if (t.ch == 0) *reinterpret_cast<float2*>(row + 2 * (t.rsub + 8 * p)) = make_float2(m1[p], m2[p]);
    }
  }
  lds_barrier();
  reinterpret_cast<float*>(own + kBwdMeans)[2 * (t.lane & 31) + (t.lane >> 5)] =
      sum_over_strips(s_row + (t.lane & 31) * 2 + (t.lane >> 5), a.strips) * a.inv_cols;
  wave_lds_fence();

  const SplitLane<PARTS> s(place.part, t.lane);
  const bool ok = t.c0 + 16 * s.chunk < a.cols;
  const int col = ok ? t.c0 + 16 * s.chunk : t.c0;
  const float sx = *reinterpret_cast<const float*>(own + kBwdScaleX + 4 * s.chunk), sg = *reinterpret_cast<const float*>(own + kBwdScaleG + 4 * s.chunk);
  float gm[16];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const float4 v = *reinterpret_cast<const float4*>(s_gamma + 16 * s.chunk + 4 * d);
    gm[4 * d] = v.x, gm[4 * d + 1] = v.y, gm[4 * d + 2] = v.z, gm[4 * d + 3] = v.w;
  }
  float y[s.PASSES][16], cg[16], cb[16];   // cg, cb: sums of g xhat and g, in units of g's block scale
#pragma unroll
  for (int p = 0; p < s.PASSES; ++p) {
    const int r = s.row0 + s.PASS_ROWS * p;
    const float rs = reinterpret_cast<const float*>(own + kBwdRstd)[r], kx = sx * rs, cx = -reinterpret_cast<const float*>(own + kBwdMean)[r] * rs;
    const float2 q = reinterpret_cast<const float2*>(own + kBwdMeans)[r];
    const float kxm = -rs * q.y * kx, krow = -rs * __builtin_fmaf(cx, q.y, q.x), rsg = rs * sg;
    const uint4 px = *reinterpret_cast<const uint4*>(own + 128 * r + 16 * s.chunk), pg = *reinterpret_cast<const uint4*>(own + kBwdG + 128 * r + 16 * s.chunk);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      float xc[4], gc[4];
      unpack4(dword_of(px, d), xc);
      unpack4(dword_of(pg, d), gc);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[p][4 * d + e] = __builtin_fmaf(xc[e], kxm, __builtin_fmaf(gc[e] * gm[4 * d + e], rsg, krow));
        if (!COLUMNS) continue;
        const float xh = __builtin_fmaf(xc[e], kx, cx);
        cg[4 * d + e] = p == 0 ? gc[e] * xh : __builtin_fmaf(gc[e], xh, cg[4 * d + e]);
        cb[4 * d + e] = p == 0 ? gc[e] : cb[4 * d + e] + gc[e];
      }
    }
  }
  store_part_of_strip<PARTS>(y, s, t.lane, ok, col, (int64_t)g * 32, a.cols, a.dX, a.SdX);
  if constexpr (COLUMNS) {
    static_assert(PARTS == 2, "a chunk belongs to the lanes that differ in bits 1 to 4");
    const float sum_g = reduce_sixteen_rows(cg, t.lane) * sg, sum_b = reduce_sixteen_rows(cb, t.lane) * sg;
    if (ok) {
      float* const dst = a.partials + (int64_t)g * 2 * a.cols + col + ((t.lane >> 1) & 15);
      store_out(dst, sum_g);
      store_out(dst + a.cols, sum_b);
    }
  }
}

// ------------------------------------------------------------------------------------------------ host
template <bool PARTIALS, int PARTS>
static void launch_split(const LayerNormRows& a, hipStream_t st) {
  launch_rows<layernorm_split_kernel<PARTIALS, PARTS>>(kFwdRowBytes + kFwdWaveBytes, split_grid<PARTS>(a.rows / 32), a.strips, a, st);
}

void launch_layernorm_split(LayerNormRows a, hipStream_t st) {
  a.strips = (a.cols + 127) / 128;
  a.teams = 1;
  a.inv_cols = 1.0 / (double)a.cols;
  a.inv_blocks = 1.0 / (double)(a.cols / 32);
  const bool four = layernorm_split_parts(a.rows, a.cols, false) == 4;
  if (a.row_mean) four ? launch_split<true, 4>(a, st) : launch_split<true, 2>(a, st);
  else four ? launch_split<false, 4>(a, st) : launch_split<false, 2>(a, st);
}

// Workgroups of at least eight waves for the sake of those that own columns (1056 x 160, whose rows need two: with four waves 5.8 us, eight
// 4.55, sixteen 4.75).  Returns the number of partial rows of dgamma | dbeta left in `partials`, 0 if it has written dgamma and dbeta.
int launch_layernorm_bwd_split(LayerNormBwdRows a, hipStream_t st) {
  a.strips = (a.cols + 127) / 128;
  a.teams = 1;
  a.inv_cols = 1.0f / (float)a.cols;
  constexpr size_t BYTES = kBwdRowBytes + kBwdWaveBytes;
  static_assert(BYTES >= 64 * sizeof(float), "the column workgroups' sums, 64 a wave");
  if (layernorm_split_columns(a.rows, a.cols)) {
    a.row_wgs = split_grid<2>(a.rows / 32);
    launch_rows<layernorm_bwd_split_kernel<2, true>>(BYTES, a.row_wgs, a.strips, a, st);
    return a.rows / 32;
  }
  const bool four = layernorm_split_parts(a.rows, a.cols, true) == 4;
  a.row_wgs = four ? split_grid<4>(a.rows / 32) : split_grid<2>(a.rows / 32);
  const int waves = std::max(a.strips, 8), grid = a.row_wgs + a.cols / 32;
  four ? launch_rows<layernorm_bwd_split_kernel<4, false>>(BYTES, grid, waves, a, st) : launch_rows<layernorm_bwd_split_kernel<2, false>>(BYTES, grid, waves, a, st);
  return 0;
}

}  // namespace jf
