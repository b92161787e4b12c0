// LayerNorm in one pass over the operands (App. A): each code is read once and written once.
//
// Bound by HBM: 2 bytes per element forward, 3 backward.  What a row needs as a whole (its moments; backward, the two row
// means) makes an operator on tiles read its operands twice; here a workgroup owns 32 whole rows, one wave per strip of
// 32 x 128 (Strip32's lane mapping), so the strip's codes stay in registers while the row sums go over the waves through
// LDS.  At block sizes 64 and 128 two or four such teams of waves own the row groups of a block row and exchange the block
// max-abs as well.  What made that slow before was that a workgroup in its arithmetic had nothing in flight.  Now workgroups are
// persistent and a wave requests the strip of its NEXT row group with direct-to-LDS loads as soon as it has moved the
// current one from LDS to registers: 4 KB (8 KB backward) per wave are in flight through all of the arithmetic, without
// registers to land in.
//
// Order of a wave's memory operations, per row group: codes LDS -> registers; request the next group into the same LDS;
// sums, workgroup barrier, results; wait for ALL its loads; only then store the results.  The wait therefore never
// includes the stores just made (loads and stores count in one counter and may finish out of order), only those of the
// previous group, which are long done.
//
// 1 M x 768, back to back: forward 446 -> 315 us (5.1 TB/s), backward with its column sums 784 -> 502 us (4.8 TB/s; vector ALU and memory
// both near their limits: 19 instructions per element) against the two-kernel scheme of jf_layernorm.hip, which stays for rows of which a
// compute unit's registers (128 per lane: 16 waves) do not hold a block row.
#pragma once
#include <algorithm>

#include "jf_layernorm.hpp"

namespace jf {

// 16 bytes per lane at a scalar base and a 32-bit lane offset (see store_out, store_as)
template <StorePolicy SP>
__device__ __forceinline__ void store_as_at(int8_t* uniform_base, uint32_t off, v4i v) {
  typedef __attribute__((address_space(1))) int8_t* gbl_ptr;
  typedef __attribute__((address_space(1))) v4i* gbl_v4i;
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  const gbl_ptr p = (gbl_ptr)uniform_base + off;
  if constexpr (SP == kStoreThrough) __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) v4u*)p, __builtin_bit_cast(v4u, v), "agent");
  else if constexpr (SP == kStoreStream) __builtin_nontemporal_store(v, (gbl_v4i)p);
  else *(gbl_v4i)p = v;
}

// A wave's place: workgroups hold `teams` teams of `strips` waves; a team owns a group of 32 rows.
struct RowWave {
  int lane, ch, rsub, wave, waves, team, strip;
  int c0, col;   // first column of the strip, of the lane's chunks (lanes outside the matrix: the strip's first chunk)
  bool ok;       // the lane's chunks lie inside the matrix
  __device__ __forceinline__ RowWave(int cols, int layout) {
    const int strips = layout & 255;
    lane = threadIdx.x & 63;
    ch = lane & 7;
    rsub = lane >> 3;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    waves = layout >> 16;
    team = wave / strips;
    strip = wave - team * strips;
    c0 = strip * 128;
    ok = c0 + 16 * ch < cols;
    col = ok ? c0 + 16 * ch : c0;
  }
  // first lane of a block, in the first of the teams that share it
  template <int B>
  __device__ __forceinline__ bool owns_scale() const { return (lane & (56 | (B / 16 - 1))) == 0 && (B == 32 || team % (B / 32) == 0); }
};

// Max-abs of the lane's block: over the lanes of a block column, then over the teams of a block row through LDS, by way of
// `at` in each wave's own part (`parts`, `part_bytes` each), which its owner has read and writes again behind the next
// barrier at the earliest.
template <int B>
__device__ __forceinline__ float block_row_max(float m, const RowWave& t, int strips, int8_t* parts, int part_bytes, int at) {
  m = wave_group_max<56 | (B / 16 - 1)>(m);
  if constexpr (B > 32) {
    constexpr int BT = B / 32;
    const auto slot = [&](int wave) { return reinterpret_cast<float*>(parts + wave * part_bytes + at) + t.ch / (B / 16); };
    wave_lds_fence();
    if ((t.lane & (56 | (B / 16 - 1))) == 0) *slot(t.wave) = m;
    lds_barrier();
#pragma unroll
    for (int k = 0; k < BT; ++k) m = fmaxf(m, *slot((t.team / BT * BT + k) * strips + t.strip));
  }
  return m;
}

// LDS of a forward wave: codes, block scales, row partials of the Add, gamma, beta, the rows' mean and rstd
constexpr int kFwdScale = 4096, kFwdPart = kFwdScale + 256, kFwdGamma = kFwdPart + 1024, kFwdBeta = kFwdGamma + 512,
              kFwdStat = kFwdBeta + 512, kFwdWaveBytes = kFwdStat + 256;
constexpr int kFwdRowBytes = 2 * 32 * 16;   // per wave: two copies (alternate row groups) of a sum pair for each of 32 rows

template <int B, bool PARTIALS, StorePolicy SP>
__global__ void __launch_bounds__(1024) layernorm_rows_kernel(const int8_t* X, const float* SX, const float* first_in, const float* second_in, int rows, int cols,
                                                              int layout, int wgs, const LayerNormRows) {
  extern __shared__ __align__(16) int8_t smem[];
  LayerNormRows a = first_arguments<PARTIALS>(X, SX, first_in, second_in, rows, cols, layout);
  const RowWave t(a.cols, layout);
  double* const s_row = reinterpret_cast<double*>(smem);                       // [copy][wave][row][sum]
  int8_t* const own = smem + t.waves * kFwdRowBytes + t.wave * kFwdWaveBytes;
  constexpr int BT = B / 32, NBC = 128 / B;            // teams of a block row, block columns of a strip
  const int groups = a.rows / 32, lc = a.cols / B;
  const uint32_t off = (uint32_t)(t.rsub * a.cols + t.col), off_scale = (uint32_t)(t.col / B) * 4;

  auto request = [&](int g) __attribute__((always_inline)) {
    const int8_t* const x = uniform_pointer(a.X + (int64_t)g * 32 * a.cols);
#pragma unroll
    for (int p = 0; p < 4; ++p) load_lds_16(x + (int64_t)p * 8 * a.cols, off, own, 1024 * p);
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SX + (int64_t)(g / BT) * lc)), off_scale, own, kFwdScale);
    if (PARTIALS) {   // the strip's block columns x 32 rows of both partials
#pragma unroll
      for (int i = 0; i < (NBC + 1) / 2; ++i) {
        const int64_t o = (int64_t)min(NBC * t.strip + 2 * i + (t.lane >> 5), lc - 1) * a.rows + g * 32 + (t.lane & 31);
        load_lds_4_vaddr(a.row_mean + o, own, kFwdPart + 256 * i);
        load_lds_4_vaddr(a.row_sumsq + o, own, kFwdPart + 512 + 256 * i);
      }
    }
  };

  int first = blockIdx.x * a.teams;                    // first row group of the workgroup's teams
  const int stride = wgs * a.teams;
  request(min(first + t.team, groups - 1));
  other_arguments<PARTIALS>(a);
  float* const s_gamma = reinterpret_cast<float*>(own + kFwdGamma);
  float* const s_beta = reinterpret_cast<float*>(own + kFwdBeta);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = t.c0 + t.lane + 64 * i;
    s_gamma[t.lane + 64 * i] = c < a.cols ? a.gamma[c] : 0.0f;
    s_beta[t.lane + 64 * i] = c < a.cols ? a.beta[c] : 0.0f;
  }
  wait_all_loads();
  wave_lds_fence();

  int copy = 0;
  for (; first < groups; first += stride, copy ^= 1) {
    const int g = first + t.team;                      // past the last group: a repeat of it that stores nothing
    uint4 px[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) px[p] = *reinterpret_cast<const uint4*>(own + 1024 * p + 16 * t.lane);
    const float sx = *reinterpret_cast<const float*>(own + kFwdScale + 4 * t.lane);
    double* const row = s_row + ((copy * t.waves + t.wave) * 32) * 2;
    if (PARTIALS) {
      const float* part = reinterpret_cast<const float*>(own + kFwdPart) + 128 * (t.lane >> 5) + (t.lane & 31);
      double v = 0.0;
#pragma unroll
      for (int j = 0; j < NBC; ++j) v += NBC * t.strip + j < lc ? (double)part[32 * j] : 0.0;
      row[2 * (t.lane & 31) + (t.lane >> 5)] = v;
    }
    wait_lds();                                        // the strip is in registers: its LDS may be filled again
    if (first + stride < groups) request(min(g + stride, groups - 1));
    if (!PARTIALS) {
      // exact integer moments of the chunk, of the block's two chunks, then in double over the strip's four blocks
      const double sd = t.ok ? (double)sx : 0.0, sd2 = sd * sd;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        int s1, s2;
        chunk_moments(px[p], s1, s2);
        s1 += lane_xor_i32<0>(s1);
        s2 += lane_xor_i32<0>(s2);
        double s = sd * (double)s1, q = sd2 * (double)s2;
        s += lane_xor_f64<1>(s);
        q += lane_xor_f64<1>(q);
        s += lane_xor_f64<2>(s);
        q += lane_xor_f64<2>(q);
        if (t.ch == 0) *reinterpret_cast<double2*>(row + 2 * (t.rsub + 8 * p)) = make_double2(s, q);
      }
    }
    lds_barrier();
    // Every wave finishes the sums of its team's 32 rows: lanes 0..31 the first sum of row lane, lanes 32..63 the second
    {
      const double* v = s_row + ((copy * t.waves + t.team * a.strips) * 32 + (t.lane & 31)) * 2 + (t.lane >> 5);
      const double sum = sum_over_strips(v, a.strips);
      const double other = lane_xor_f64<5>(sum);
      const double mud = (t.lane < 32 ? sum : other) * (PARTIALS ? a.inv_blocks : a.inv_cols);
      const float var = fmaxf((float)((t.lane < 32 ? other : sum) * a.inv_cols - mud * mud), 0.0f);
      const float ve = var + a.eps;
      float rs = __builtin_amdgcn_rsqf(ve);            // refined by one Newton step (relative error about 1e-7)
      rs = rs * __builtin_fmaf(-0.5f * ve * rs, rs, 1.5f);
      if (t.lane < 32) reinterpret_cast<float2*>(own + kFwdStat)[t.lane] = make_float2((float)mud, rs);
      wave_lds_fence();
      if (t.strip == 0 && t.lane < 32 && g < groups) {
        // (stores: counted with the loads, hence before the wait below, not before the next group's)
        a.mean[g * 32 + t.lane] = (float)mud;
        a.rstd[g * 32 + t.lane] = rs;
      }
    }
    float k1[4], kb[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float2 st = reinterpret_cast<const float2*>(own + kFwdStat)[t.rsub + 8 * p];
      k1[p] = sx * st.y;
      kb[p] = __builtin_fmaf(-128.0f, k1[p], -st.x * st.y);
    }
    float y[4][16];
    float m = 0.0f;
#pragma unroll
    for (int d = 0; d < 4; ++d) {                      // four columns at a time: gamma and beta come out of LDS
      const float4 gm = *reinterpret_cast<const float4*>(s_gamma + 16 * t.ch + 4 * d), bt = *reinterpret_cast<const float4*>(s_beta + 16 * t.ch + 4 * d);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const uint32_t w = dword_of(px[p], d) ^ 0x80808080u;   // code + 128 per byte
        y[p][4 * d + 0] = __builtin_fmaf(__builtin_fmaf((float)(w & 0xffu), k1[p], kb[p]), gm.x, bt.x);
        y[p][4 * d + 1] = __builtin_fmaf(__builtin_fmaf((float)((w >> 8) & 0xffu), k1[p], kb[p]), gm.y, bt.y);
        y[p][4 * d + 2] = __builtin_fmaf(__builtin_fmaf((float)((w >> 16) & 0xffu), k1[p], kb[p]), gm.z, bt.z);
        y[p][4 * d + 3] = __builtin_fmaf(__builtin_fmaf((float)(w >> 24), k1[p], kb[p]), gm.w, bt.w);
      }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) m = amax16(m, y[p]);
    m = block_row_max<B>(m, t, a.strips, smem + t.waves * kFwdRowBytes, kFwdWaveBytes, kFwdStat);
    float scale;
    double inv;
    block_scale(m, scale, inv);
    uint4 o[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      o[p] = quantize16(y[p], inv);
      asm volatile("" : "+v"(o[p].x), "+v"(o[p].y), "+v"(o[p].z), "+v"(o[p].w));
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_all_loads();
    if (t.ok && g < groups) {
      // uniform base + 32-bit lane offset, like the loads: no 64-bit lane addresses to keep
      int8_t* const out = uniform_pointer(a.Y + (int64_t)g * 32 * a.cols);
#pragma unroll
      for (int p = 0; p < 4; ++p) store_as_at<SP>(out + (int64_t)p * 8 * a.cols, off, v4i{(int)o[p].x, (int)o[p].y, (int)o[p].z, (int)o[p].w});
      if (t.owns_scale<B>()) store_scale<SP>(reinterpret_cast<int8_t*>(uniform_pointer(a.SY + (int64_t)(g / BT) * lc)) + off_scale, scale);
    }
  }
}

// LDS of a backward wave: codes of x and of g, their block scales, mean and rstd of the 32 rows, gamma, the two row means
constexpr int kBwdG = 4096, kBwdScaleX = 8192, kBwdScaleG = kBwdScaleX + 256, kBwdMean = kBwdScaleG + 256, kBwdRstd = kBwdMean + 128,
              kBwdGamma = kBwdRstd + 128, kBwdMeans = kBwdGamma + 512, kBwdWaveBytes = kBwdMeans + 256;
constexpr int kBwdRowBytes = 2 * 32 * 8;

// dgamma and dbeta of 32 columns straight from g and x: a lane owns 16 columns of row l % 32 of its wave's row groups.
// The column sums need nothing of the row pass, only its operands a second time, which for a short tensor come out of L2: this saves the
// launch that adds the partial rows, and the row pass 8 of its 20 instructions per element.  Bound by the lines that a compute unit
// pulls in for a quarter of each: with many rows the workgroups of the few block columns take longer than the row pass (4096 x 768 10.3
// -> 13.9 us; with 16 columns to a workgroup 16.5).
template <int B>
__device__ __forceinline__ void column_sums_direct(const LayerNormBwdRows& a, int index, int waves, float* s_sum) {
  const int lane = threadIdx.x & 63, row = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // A line of 128 columns belongs to four of these workgroups: they are on one XCD (to which workgroups come in turns), so that its L2
  // fetches the line once.
  const int columns = a.cols / 32, xcd = index & 7, group = xcd * (columns >> 3) + min(xcd, columns & 7) + (index >> 3);
  const int col = group * 32 + 16 * (lane >> 5), lc = a.cols / B;
  float sums[32];   // of g xhat, then of g
#pragma unroll
  for (int e = 0; e < 32; ++e) sums[e] = 0.0f;
  // four row groups requested together: one after the other each waits for memory by itself (2048 x 768 7.9 -> 7.65 us, and with the
  // sums over the lanes by halves 7.0)
  constexpr int AHEAD = 4;
  const int groups = a.rows / 32;
  for (int first = wave; first < groups; first += AHEAD * waves) {
    uint4 px[AHEAD], pg[AHEAD];
    float rs[AHEAD], mu[AHEAD], sx[AHEAD], sg[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      const int g = min(first + i * waves, groups - 1);
      const int64_t at = (int64_t)(g * 32 + row) * a.cols + col, block = (int64_t)(g / (B / 32)) * lc + group / (B / 32);
      px[i] = *reinterpret_cast<const uint4*>(a.X + at);
      pg[i] = *reinterpret_cast<const uint4*>(a.G + at);
      rs[i] = a.rstd[g * 32 + row];
      mu[i] = a.mean[g * 32 + row];
      sx[i] = a.SX[block];
      sg[i] = a.SG[block];
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      if (first + i * waves >= groups) break;   // the same for the whole wave
      const float kx = sx[i] * rs[i], cx = -mu[i] * rs[i];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        float x[4], gr[4];
        unpack4(dword_of(px[i], d), x);
        unpack4(dword_of(pg[i], d), gr);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gv = gr[e] * sg[i];
          sums[4 * d + e] = __builtin_fmaf(gv, __builtin_fmaf(x[e], kx, cx), sums[4 * d + e]);
          sums[16 + 4 * d + e] += gv;
        }
      }
    }
  }
  const int value = reduce_rows_of_32(sums, lane);
  s_sum[64 * wave + 32 * (value >> 4) + 16 * (lane >> 5) + (value & 15)] = sums[0];
  __syncthreads();
  if (threadIdx.x < 64) {   // the waves in order
    double v = 0.0;
    for (int w = 0; w < waves; ++w) v += (double)s_sum[64 * w + lane];
    (lane < 32 ? a.dgamma : a.dbeta)[group * 32 + row] = (float)v;
  }
}

// dx = rstd (ghat - mean_C(ghat) - xhat mean_C(ghat xhat)) with ghat = g gamma, xhat = (x - mean) rstd; the column sums
// of g xhat and g stay in registers over all row groups and end as one partial row of dgamma | dbeta per workgroup.
// COLUMNS_APART: the column sums are left to workgroups of their own behind the row_wgs that own rows (column_sums_direct).
// KEPT: of how many of a lane's four rows ghat stays in registers between the two passes over the strip, 16 each, instead of
// being formed again (two instructions per element).  Workgroups of at most 12 waves, three on a SIMD, have 168 registers: room
// for two rows beside the column sums, for all four without them; 16 waves have none.  More than fits goes to scratch
// memory, whose loads also wait for the strips in flight (1 M x 768 on the day of the choice, kernel alone, three rows 513 us, two 484, one 515,
// none 535; two now 486 to 514 in a trace).
template <int B, StorePolicy SP, bool COLUMNS_APART, int KEPT>
__global__ void __launch_bounds__(KEPT ? 768 : 1024) layernorm_bwd_rows_kernel(
    const int8_t* G, const float* SG, const int8_t* X, const float* SX, int rows, int cols, int layout, int wgs, const float* gamma, const LayerNormBwdRows) {
  extern __shared__ __align__(16) int8_t smem[];
  LayerNormBwdRows a = first_arguments(G, SG, X, SX, rows, cols, layout, wgs, gamma);
  // A bound on the strips would keep the compiler from unrolling the sums over them, which here, unlike forward, is the faster way
  // (147648 x 1120 137.0 -> 136.0 us, 1 M x 768 514 -> 512; at block 128 it takes the registers that there are not).
  if constexpr (B == 32) asm("" : "+s"(a.strips));
  if (COLUMNS_APART && (int)blockIdx.x >= a.row_wgs) {
    other_arguments(a);
    column_sums_direct<B>(a, blockIdx.x - a.row_wgs, layout >> 16, reinterpret_cast<float*>(smem));
    return;
  }
  const RowWave t(a.cols, layout);
  float* const s_row = reinterpret_cast<float*>(smem);                         // [copy][wave][row][sum]
  int8_t* const own = smem + t.waves * kBwdRowBytes + t.wave * kBwdWaveBytes;
  constexpr int BT = B / 32, NBC = 128 / B;            // teams of a block row, block columns of a strip
  const int groups = a.rows / 32, lc = a.cols / B;
  const uint32_t off = (uint32_t)(t.rsub * a.cols + t.col), off_scale = (uint32_t)(t.col / B) * 4;

  auto request_codes = [&](int g) __attribute__((always_inline)) {
    const int8_t* const x = uniform_pointer(a.X + (int64_t)g * 32 * a.cols);
    const int8_t* const gr = uniform_pointer(a.G + (int64_t)g * 32 * a.cols);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      load_lds_16(x + (int64_t)p * 8 * a.cols, off, own, 1024 * p);
      load_lds_16(gr + (int64_t)p * 8 * a.cols, off, own, kBwdG + 1024 * p);
    }
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SX + (int64_t)(g / BT) * lc)), off_scale, own, kBwdScaleX);
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SG + (int64_t)(g / BT) * lc)), off_scale, own, kBwdScaleG);
  };
  auto request_stats = [&](int g) __attribute__((always_inline)) {
    if (t.lane < 32) {   // 32 floats each
      load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.mean + g * 32)), (uint32_t)t.lane * 4, own, kBwdMean);
      load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.rstd + g * 32)), (uint32_t)t.lane * 4, own, kBwdRstd);
    }
  };

  int first = blockIdx.x * a.teams;
  const int stride = a.row_wgs * a.teams;
  request_codes(min(first + t.team, groups - 1));
  other_arguments(a);
  request_stats(min(first + t.team, groups - 1));
  float* const s_gamma = reinterpret_cast<float*>(own + kBwdGamma);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = t.c0 + t.lane + 64 * i;
    s_gamma[t.lane + 64 * i] = c < a.cols ? a.gamma[c] : 0.0f;
  }
  wait_all_loads();
  wave_lds_fence();

  float cgs[16], cbs[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) cgs[e] = cbs[e] = 0.0f;
  int copy = 0;
  for (; first < groups; first += stride, copy ^= 1) {
    const int g = first + t.team;                      // past the last group: a repeat of it that adds and stores nothing
    uint4 px[4], pg[4];
    float mu[4], rs[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      px[p] = *reinterpret_cast<const uint4*>(own + 1024 * p + 16 * t.lane);
      pg[p] = *reinterpret_cast<const uint4*>(own + kBwdG + 1024 * p + 16 * t.lane);
      mu[p] = reinterpret_cast<const float*>(own + kBwdMean)[t.rsub + 8 * p];
      rs[p] = reinterpret_cast<const float*>(own + kBwdRstd)[t.rsub + 8 * p];
    }
    const float sx = *reinterpret_cast<const float*>(own + kBwdScaleX + 4 * t.lane);
    float sg = *reinterpret_cast<const float*>(own + kBwdScaleG + 4 * t.lane);
    wait_lds();                                        // the strips are in registers: their LDS may be filled again
    if (first + stride < groups) request_codes(min(g + stride, groups - 1)), request_stats(min(g + stride, groups - 1));
    sg = t.ok && g < groups ? sg : 0.0f;               // what lies outside adds nothing to the sums
    float kx[4], cx[4], m1[4], m2[4];
    float y[4][16];                                    // dx; ghat in units of g's block scale before, of KEPT rows
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      kx[p] = sx * rs[p];
      cx[p] = -mu[p] * rs[p];                          // xhat = code kx + cx
      m1[p] = m2[p] = 0.0f;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const float4 gm4 = *reinterpret_cast<const float4*>(s_gamma + 16 * t.ch + 4 * d);
      const float gm[4] = {gm4.x, gm4.y, gm4.z, gm4.w};
      // g in units of its block scale, which goes onto the sums of the four rows instead of onto every element
      float tg[4], tb[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float x[4], gr[4];
        unpack4(dword_of(px[p], d), x);
        unpack4(dword_of(pg[p], d), gr);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float xh = __builtin_fmaf(x[e], kx[p], cx[p]), gh = gr[e] * gm[e];
          if (p < KEPT) y[p][4 * d + e] = gh;
          // in place (left to itself the compiler keeps the operands of many deferred updates alive instead)
          asm volatile("v_add_f32 %0, %0, %1" : "+v"(m1[p]) : "v"(gh));
          asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(m2[p]) : "v"(gh), "v"(xh));
          if (COLUMNS_APART) continue;
          tg[e] = p == 0 ? gr[e] * xh : __builtin_fmaf(gr[e], xh, tg[e]);
          if (p == 0) tb[e] = gr[e];
          else asm volatile("v_add_f32 %0, %0, %1" : "+v"(tb[e]) : "v"(gr[e]));
        }
        __builtin_amdgcn_sched_barrier(0);             // interleaved passes would keep their unpacked values live together
      }
#pragma unroll
      for (int e = 0; e < 4 && !COLUMNS_APART; ++e) {
        asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(cgs[4 * d + e]) : "v"(sg), "v"(tg[e]));
        asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(cbs[4 * d + e]) : "v"(sg), "v"(tb[e]));
      }
    }
    float* const row = s_row + ((copy * t.waves + t.wave) * 32) * 2;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      m1[p] = wave_group_sum<7>(m1[p] * sg);
      m2[p] = wave_group_sum<7>(m2[p] * sg);
      if (t.ch == 0) *reinterpret_cast<float2*>(row + 2 * (t.rsub + 8 * p)) = make_float2(m1[p], m2[p]);
    }
    lds_barrier();
    {
      const float* v = s_row + ((copy * t.waves + t.team * a.strips) * 32 + (t.lane & 31)) * 2 + (t.lane >> 5);
      reinterpret_cast<float*>(own + kBwdMeans)[2 * (t.lane & 31) + (t.lane >> 5)] = sum_over_strips(v, a.strips) * a.inv_cols;
      wave_lds_fence();
    }
    // the codes are unpacked again below: 128 floats kept from above would not fit the registers of three waves per SIMD
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      asm volatile("" : "+v"(px[p].x), "+v"(px[p].y), "+v"(px[p].z), "+v"(px[p].w));
      asm volatile("" : "+v"(pg[p].x), "+v"(pg[p].y), "+v"(pg[p].z), "+v"(pg[p].w));
    }
    // dx = (g_code gamma) (rstd sg) + x_code kxm + krow.  The order is part of the result: another one, as accurate, moves one code in a
    // million over a rounding tie, and with it now and then the scale of a block in the operators that take dx.
    float kxm[4], krow[4], rsg[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float2 q = reinterpret_cast<const float2*>(own + kBwdMeans)[t.rsub + 8 * p];
      kxm[p] = -rs[p] * q.y * kx[p];
      krow[p] = -rs[p] * __builtin_fmaf(cx[p], q.y, q.x);
      rsg[p] = rs[p] * sg;
    }
    float m = 0.0f;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      float gm[4];
      if constexpr (KEPT < 4) {
        const float4 gm4 = *reinterpret_cast<const float4*>(s_gamma + 16 * t.ch + 4 * d);
        gm[0] = gm4.x, gm[1] = gm4.y, gm[2] = gm4.z, gm[3] = gm4.w;
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float x[4], gr[4];
        unpack4(dword_of(px[p], d), x);
        if (p >= KEPT) unpack4(dword_of(pg[p], d), gr);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          y[p][4 * d + e] = __builtin_fmaf(x[e], kxm[p], __builtin_fmaf(p < KEPT ? y[p][4 * d + e] : gr[e] * gm[e], rsg[p], krow[p]));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) m = amax16(m, y[p]);
    m = block_row_max<B>(m, t, a.strips, smem + t.waves * kBwdRowBytes, kBwdWaveBytes, kBwdMeans);
    float scale;
    double inv;
    block_scale(m, scale, inv);
    uint4 o[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      o[p] = quantize16(y[p], inv);
      asm volatile("" : "+v"(o[p].x), "+v"(o[p].y), "+v"(o[p].z), "+v"(o[p].w));
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_all_loads();
    if (t.ok && g < groups) {
      // uniform base + 32-bit lane offset, like the loads: no 64-bit lane addresses to keep
      int8_t* const out = uniform_pointer(a.dX + (int64_t)g * 32 * a.cols);
#pragma unroll
      for (int p = 0; p < 4; ++p) store_as_at<SP>(out + (int64_t)p * 8 * a.cols, off, v4i{(int)o[p].x, (int)o[p].y, (int)o[p].z, (int)o[p].w});
      if (t.owns_scale<B>()) store_scale<SP>(reinterpret_cast<int8_t*>(uniform_pointer(a.SdX + (int64_t)(g / BT) * lc)) + off_scale, scale);
    }
  }

  if (COLUMNS_APART) return;
  // column sums over the 8 row lanes of the wave, then over the teams through LDS, in a fixed order
  float sums[8];
  reduce_rows32(cgs, cbs, sums);
  const int place = reduced_column(t.lane);            // + j % 4: dgamma for j < 4, dbeta beyond
  if (a.teams > 1) {
    float* const mine = reinterpret_cast<float*>(own);   // all requests have landed and nobody else uses this wave's part
#pragma unroll
    for (int j = 0; j < 8; ++j) mine[128 * (j / 4) + j % 4 + place] = sums[j];   // (twice, by lanes 8 apart)
    lds_barrier();
    if (t.team == 0) {
      for (int k = 1; k < a.teams; ++k) {
        const float* other = reinterpret_cast<const float*>(own + k * a.strips * kBwdWaveBytes);
#pragma unroll
        for (int j = 0; j < 8; ++j) sums[j] += other[128 * (j / 4) + j % 4 + place];
      }
    }
  }
  if (t.team == 0 && t.ok && (t.lane & 8) == 0) store_partials(a.partials + (int64_t)blockIdx.x * 2 * a.cols + t.c0 + place, a.cols, sums);
}

// ------------------------------------------------------------------------------------------------ host
// A launch needs more LDS than a kernel gets by default.  The limit belongs to the kernel on the current device, so it is
// raised in front of every launch (0.07 us) instead of once; where it cannot be, nothing is launched and launch_status()
// reports the error.
template <auto KERNEL>
static bool raise_lds(size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
}
inline int rows_layout(int strips, int teams, int waves) { return strips | teams << 8 | waves << 16; }
template <auto KERNEL>
static void launch_rows(size_t wave_bytes, int grid, int waves, const LayerNormRows& a, hipStream_t st) {
  typedef KernelParameters<decltype(KERNEL)> Parameters;
  static_assert(Parameters::template preloaded<7>() && Parameters::template stands_at<8, LayerNormRows>(offsetof(LayerNormRowsArgs, all)), "LayerNormRowsArgs");
  if (!raise_lds<KERNEL>(16 * wave_bytes)) return;
  hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(64 * waves), waves * wave_bytes, st, a.X, a.SX, a.row_mean ? a.row_mean : a.gamma,
                     a.row_mean ? a.row_sumsq : a.beta, a.rows, a.cols, rows_layout(a.strips, a.teams, waves), grid, a);
}
template <auto KERNEL>
static void launch_rows(size_t wave_bytes, int grid, int waves, const LayerNormBwdRows& a, hipStream_t st) {
  typedef KernelParameters<decltype(KERNEL)> Parameters;
  static_assert(Parameters::template preloaded<8>() && Parameters::template stands_at<9, LayerNormBwdRows>(offsetof(LayerNormBwdRowsArgs, all)), "LayerNormBwdRowsArgs");
  if (!raise_lds<KERNEL>(16 * wave_bytes)) return;
  hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(64 * waves), waves * wave_bytes, st, a.G, a.SG, a.X, a.SX, a.rows, a.cols,
                     rows_layout(a.strips, a.teams, waves), a.row_wgs, a.gamma, a);
}

// Teams per workgroup, one workgroup per compute unit.  The waves of a workgroup are dealt to the four SIMDs in turn, so
// that the fullest SIMD sets the pace: the count that does most row groups per wave of that SIMD (six strips: two teams, 3
// waves on every SIMD, instead of two workgroups of one team, which leave 2, 3, 3 and 4: 622 -> 571 us backward at 1 M x
// 768), of equal ones the larger; fewer while there are compute units without a workgroup.  Whole block rows: `step` teams.
static int choose_teams(int strips, int groups, int step) {
  int best = step;
  for (int n = 2 * step; n * strips <= 16; n += step)
    if ((n * strips + 3) / 4 * best <= (best * strips + 3) / 4 * n) best = n;
  return std::max(step, std::min(best, (groups / step + 255) / 256 * step));
}

template <int B>
static void launch_layernorm_rows_b(LayerNormRows a, hipStream_t st) {
  const int groups = a.rows / 32;
  a.strips = (a.cols + 127) / 128;
  a.teams = choose_teams(a.strips, groups, B / 32);
  a.inv_cols = 1.0 / (double)a.cols;
  a.inv_blocks = 1.0 / (double)(a.cols / B);
  const int waves = a.strips * a.teams, grid = std::min((groups + a.teams - 1) / a.teams, 256);
  with_store_policy(a.rows, a.cols, [&](auto sp) {
    if (a.row_mean) launch_rows<layernorm_rows_kernel<B, true, decltype(sp)::value>>(kFwdRowBytes + kFwdWaveBytes, grid, waves, a, st);
    else launch_rows<layernorm_rows_kernel<B, false, decltype(sp)::value>>(kFwdRowBytes + kFwdWaveBytes, grid, waves, a, st);
  });
}

template <int B>
static int launch_layernorm_bwd_rows_b(LayerNormBwdRows a, bool in_place, hipStream_t st) {
  const int groups = a.rows / 32;
  a.strips = (a.cols + 127) / 128;
  a.teams = choose_teams(a.strips, groups, B / 32);
  a.inv_cols = 1.0f / (float)a.cols;
  const int waves = a.strips * a.teams;
  a.row_wgs = std::min((groups + a.teams - 1) / a.teams, 256);
  static_assert(16 * (kBwdRowBytes + kBwdWaveBytes) <= 160 * 1024, "sixteen waves share the LDS of a compute unit");
  const bool apart = B > 32 && !in_place && a.rows <= 2048 && groups <= 12 * waves;   // at most 12 row groups for a wave of the column workgroups
  constexpr size_t BYTES = kBwdRowBytes + kBwdWaveBytes;
  with_store_policy(a.rows, a.cols, [&](auto sp) {
    constexpr StorePolicy SP = decltype(sp)::value;
    if constexpr (SP == kStoreThrough && B > 32) {   // (2048 rows are always stored through; block size 32: jf_layernorm_split.hip)
      if (apart) {
        const int grid = a.row_wgs + a.cols / 32;
        if (waves <= 12) launch_rows<layernorm_bwd_rows_kernel<B, SP, true, 4>>(BYTES, grid, waves, a, st);
        else launch_rows<layernorm_bwd_rows_kernel<B, SP, true, 0>>(BYTES, grid, waves, a, st);
        return;
      }
    }
    if (waves <= 12) launch_rows<layernorm_bwd_rows_kernel<B, SP, false, 2>>(BYTES, a.row_wgs, waves, a, st);
    else launch_rows<layernorm_bwd_rows_kernel<B, SP, false, 0>>(BYTES, a.row_wgs, waves, a, st);
  });
  return apart ? 0 : a.row_wgs;
}

// One translation unit per block size instantiates the launches, so that the kernels compile in parallel.
#define JF_LAYERNORM_ROWS_INSTANCE(B)                                                                            \
  namespace jf {                                                                                                 \
  void launch_layernorm_rows_b##B(const LayerNormRows& a, hipStream_t st) { launch_layernorm_rows_b<B>(a, st); } \
  int launch_layernorm_bwd_rows_b##B(const LayerNormBwdRows& a, bool in_place, hipStream_t st) {                 \
    return launch_layernorm_bwd_rows_b<B>(a, in_place, st);                                                      \
  }                                                                                                              \
  }

}  // namespace jf
