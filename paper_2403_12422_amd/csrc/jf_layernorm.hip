// INT8-in / INT8-out LayerNorm, forward and backward (App. A).
//
// Rows of at most 2048 / 1024 / 512 columns at block size 32 / 64 / 128 go through jf_layernorm_rows.hpp where there are enough
// of them (layernorm_rows_fits), wider ones at block size 32 through jf_layernorm_wide.hip (layernorm_wide_fits).  Otherwise each
// pass is a small kernel that only leaves sums (row statistics forward; row means and dgamma | dbeta partial rows backward) followed by an
// element-wise operator on tiles: the 32 x 128 strips of jf_rowops.hpp at block size 32, workgroups of B rows x 128
// columns at block sizes 64 and 128.  No workgroup holds a row in registers, so rows may be of any width.
// Row sums of the forward pass come from exact integer dot products of the codes (v_dot4), scaled per block -- the
// row-partials scheme of App. A applied to the INT8 input itself -- or from the partials that the preceding Add wrote.
#include <algorithm>
#include <mutex>

#include "jf_layernorm.hpp"

namespace jf {

// ------------------------------------------------------------------------------------------------
// The backward sums kernel: a workgroup owns 32 whole rows at a time (at every block size: a block row is one, two or four such
// groups) and is made of strip waves: wave w holds the 32 x 128 strip w of those rows with the lane mapping of Strip32
// (C / 128 waves, at most 16).  What needs a whole row (the row sums) is reduced over the 8 chunk lanes of a row inside each wave (three DPP steps)
// and over the strips through a few hundred bytes of LDS, in a fixed order; what belongs to a column (gamma, the column sums)
// never leaves its wave.
struct RowStrips {
  int ch, rsub, wave, nstrips;
  int lc, col, log2b;
  bool ok;
  __device__ __forceinline__ RowStrips(int cols, int block_log2, int strips) {
    const int lane = threadIdx.x & 63;
    ch = lane & 7;
    rsub = lane >> 3;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    nstrips = strips;
    log2b = block_log2;
    lc = cols >> log2b;
    // rows wider than 16 strips (2048 columns) are shared evenly by the workgroups blockIdx.y = 0, 1, ...
    const int c0 = (blockIdx.y * nstrips + wave) * 128, c = c0 + 16 * ch;
    ok = c < cols;
    col = ok ? c : min(c0, cols - 32);   // lanes outside the matrix point at a valid chunk instead, see Strip32
  }
  // element offset of the lane's chunk of row rsub of the 32-row group g; pass p adds 8 p cols
  __device__ __forceinline__ int64_t base(int g, int cols) const { return (int64_t)(g * 32 + rsub) * cols + col; }
  // index of the lane's quantization block in a scale grid
  __device__ __forceinline__ int64_t block_index(int g) const { return (int64_t)(g * 32 >> log2b) * lc + (col >> log2b); }
};

// Row statistics of LayerNorm from the codes (the per-row mean and sum of squares of App. A, here taken of the INT8 input
// itself), for rows of any width: the workgroup's waves share the strips of its 32 rows (wave w takes strips w, w + waves, ...).
// Per 16-code chunk the sum and the sum of squares of the codes are exact integers (v_dot4); times the block scale,
// in double, they are the chunk's share of the row's sum and sum of squares.  The shares are added over a lane's
// strips, over the 8 chunk lanes of a row (three DPP steps) and over the waves through LDS, in a fixed order.  The
// normalisation itself is an element-wise operator on strips or tiles.
__global__ void __launch_bounds__(1024) layernorm_row_stats_kernel(const int8_t* __restrict__ X, const float* __restrict__ SX,
                                                                  float eps, int rows, int cols, int block_log2, int nwaves,
                                                                  float* __restrict__ mean_out, float* __restrict__ rstd_out) {
  __shared__ double s_row[16][32][2];
  const int lane = threadIdx.x & 63, ch = lane & 7, rsub = lane >> 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bi = blockIdx.x, lc = cols >> block_log2;   // bi: group of 32 rows
  const int64_t pass = (int64_t)8 * cols;
  double cs[4] = {0.0, 0.0, 0.0, 0.0}, cq[4] = {0.0, 0.0, 0.0, 0.0};
  for (int c0 = wave * 128; c0 < cols; c0 += nwaves * 128) {
    const bool ok = c0 + 16 * ch < cols;
    const int col = ok ? c0 + 16 * ch : c0;   // lanes outside the matrix read the strip's first chunk and add nothing
    const int64_t base = (int64_t)(bi * 32 + rsub) * cols + col;
    uint4 px[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) px[p] = *reinterpret_cast<const uint4*>(X + base + p * pass);
    const double sd = ok ? (double)SX[(int64_t)(bi * 32 >> block_log2) * lc + (col >> block_log2)] : 0.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      int s1, s2;
      chunk_moments(px[p], s1, s2);
      cs[p] += sd * (double)s1;
      cq[p] += sd * sd * (double)s2;
    }
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const double s = wave_group_sum_f64<7>(cs[p]), q = wave_group_sum_f64<7>(cq[p]);
    if (ch == 0) {
      s_row[wave][rsub + 8 * p][0] = s;
      s_row[wave][rsub + 8 * p][1] = q;
    }
  }
  __syncthreads();
  if (threadIdx.x < 32) {   // row threadIdx.x of the block: the waves in a fixed order
    double s = 0.0, q = 0.0;
    for (int w = 0; w < nwaves; ++w) {
      s += s_row[w][threadIdx.x][0];
      q += s_row[w][threadIdx.x][1];
    }
    const double inv_cols = 1.0 / (double)cols, mud = s * inv_cols;
    const float var = fmaxf((float)(q * inv_cols - mud * mud), 0.0f);
    // reciprocal square root: hardware approximation refined by one Newton step (relative error ~1e-7)
    const float ve = var + eps;
    float rs = __builtin_amdgcn_rsqf(ve);
    rs = rs * __builtin_fmaf(-0.5f * ve * rs, rs, 1.5f);
    mean_out[bi * 32 + threadIdx.x] = (float)mud;
    rstd_out[bi * 32 + threadIdx.x] = rs;
  }
}

// LayerNorm backward, in two kernels.  With ghat = g gamma and xhat = (x - mean) rstd,
//   dx = rstd (ghat - mean_C(ghat) - xhat mean_C(ghat xhat)),  dgamma = sum_N g xhat,  dbeta = sum_N g.
// Everything that needs a whole row or a whole column is a sum, and sums are cheap to hand over: the first kernel
// reads g and x once and leaves the two row means per row and one row of dgamma | dbeta partial sums per workgroup
// in the workspace; the second one is an element-wise operator on tiles like GELU backward.  (One kernel
// that does both has to keep dx, the codes and the column sums in registers at once: about 250, which leaves a
// compute unit with a single workgroup and nothing to overlap its memory latency with.)
//
// First kernel: the workgroup of strip waves described above walks over the row blocks blockIdx.x, blockIdx.x +
// gridDim.x, ..., one 32 x 128 strip of each in a wave.  Ten instructions per element (the block scale of g goes onto sums, not
// onto elements; in place of fifteen, with the column reduction of jf_layernorm.hpp and even column ranges: 4096 x 2560 at block 32,
// whole pass, 19.5 -> 16.6 us, 4096 x 4096 at 64 22.6 -> 21.3, 2048 x 1024 at 128 11.1 -> 10.2).  The row sums go over the chunk
// lanes, then over the strips through LDS (two copies used by alternate row blocks: one barrier per block); the running column sums of
// g xhat and g stay in registers over all row blocks -- a lane always holds the same 16 columns -- and are added
// over the 8 row lanes of the wave at the end (every wave owns its own 128 columns of the partial row).  All orders
// are fixed: results are bit-stable from run to run.
// LDS of a wave: codes of x and of g, their block scales, mean and rstd of the 32 rows
constexpr int kSumsG = 4096, kSumsScaleX = 8192, kSumsScaleG = kSumsScaleX + 256, kSumsMean = kSumsScaleG + 256, kSumsRstd = kSumsMean + 128,
              kSumsWaveBytes = kSumsRstd + 128, kSumsRowBytes = 2 * 32 * 8;
template <bool AHEAD>
__global__ void __launch_bounds__(1024) layernorm_bwd_sums_kernel(
    const int8_t* __restrict__ G, const int8_t* __restrict__ X, const float* __restrict__ SG, const float* __restrict__ SX, int rows, int cols, int block_log2,
    int strips, const float* __restrict__ gamma, const float* __restrict__ mean_in, const float* __restrict__ rstd_in, float* __restrict__ row_means,
    float* __restrict__ partials) {
  extern __shared__ __align__(16) int8_t smem[];
  const RowStrips t(cols, block_log2, strips);
  float* const s_row = reinterpret_cast<float*>(smem);   // [row block parity][strip][row][sum of ghat, of ghat xhat]
  int8_t* const own = smem + t.nstrips * kSumsRowBytes + t.wave * kSumsWaveBytes;   // with AHEAD
  const int nblocks = rows / 32, lane = threadIdx.x & 63;
  const float inv_cols = 1.0f / (float)cols;
  const uint32_t off = (uint32_t)(t.rsub * cols + t.col), off_scale = (uint32_t)(t.col >> block_log2) * 4;
  auto request = [&](int g) __attribute__((always_inline)) {
    const int8_t* const x = uniform_pointer(X + (int64_t)g * 32 * cols);
    const int8_t* const gr = uniform_pointer(G + (int64_t)g * 32 * cols);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      load_lds_16(x + (int64_t)p * 8 * cols, off, own, 1024 * p);
      load_lds_16(gr + (int64_t)p * 8 * cols, off, own, kSumsG + 1024 * p);
    }
    const int64_t grid_row = (int64_t)(g * 32 >> block_log2) * t.lc;
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(SX + grid_row)), off_scale, own, kSumsScaleX);
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(SG + grid_row)), off_scale, own, kSumsScaleG);
    if (lane < 32) {   // 32 floats each
      load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(mean_in + g * 32)), (uint32_t)lane * 4, own, kSumsMean);
      load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(rstd_in + g * 32)), (uint32_t)lane * 4, own, kSumsRstd);
    }
  };
  if (AHEAD) request(blockIdx.x);
  float gm[16], cgs[16], cbs[16];
  load16f(gamma + t.col, gm);
#pragma unroll
  for (int e = 0; e < 16; ++e) cgs[e] = cbs[e] = 0.0f;
  if (AHEAD) wait_all_loads();

  int parity = 0;
  for (int bi = blockIdx.x; bi < nblocks; bi += gridDim.x, parity ^= 1) {
    uint4 px[4], pg[4];
    float mu[4], rs[4], sx, sg;
    if constexpr (AHEAD) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        px[p] = *reinterpret_cast<const uint4*>(own + 1024 * p + 16 * lane);
        pg[p] = *reinterpret_cast<const uint4*>(own + kSumsG + 1024 * p + 16 * lane);
        mu[p] = reinterpret_cast<const float*>(own + kSumsMean)[t.rsub + 8 * p];
        rs[p] = reinterpret_cast<const float*>(own + kSumsRstd)[t.rsub + 8 * p];
      }
      sx = *reinterpret_cast<const float*>(own + kSumsScaleX + 4 * lane);
      sg = *reinterpret_cast<const float*>(own + kSumsScaleG + 4 * lane);
      wait_lds();                                        // the strips are in registers: their LDS may be filled again
      if (bi + (int)gridDim.x < nblocks) request(bi + gridDim.x);
    } else {
      const int64_t base = t.base(bi, cols);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        px[p] = *reinterpret_cast<const uint4*>(X + base + (int64_t)p * 8 * cols);
        pg[p] = *reinterpret_cast<const uint4*>(G + base + (int64_t)p * 8 * cols);
        mu[p] = mean_in[bi * 32 + t.rsub + 8 * p];
        rs[p] = rstd_in[bi * 32 + t.rsub + 8 * p];
      }
      sx = SX[t.block_index(bi)];
      sg = SG[t.block_index(bi)];
    }
    sg = t.ok ? sg : 0.0f;                               // lanes outside the matrix add nothing to the sums
    float kx[4], cx[4], m1[4], m2[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      kx[p] = sx * rs[p];
      cx[p] = -mu[p] * rs[p];                          // xhat = code kx + cx
      m1[p] = m2[p] = 0.0f;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      // g in units of its block scale, which goes onto the sums of the four rows instead of onto every element
      float tg[4], tb[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float x[4], gr[4];
        unpack4(dword_of(px[p], d), x);
        unpack4(dword_of(pg[p], d), gr);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float xh = __builtin_fmaf(x[e], kx[p], cx[p]), gh = gr[e] * gm[4 * d + e];
          // the sums are updated in place, in program order (left to itself the compiler keeps the operands of many deferred
          // updates alive instead)
          asm volatile("v_add_f32 %0, %0, %1" : "+v"(m1[p]) : "v"(gh));
          asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(m2[p]) : "v"(gh), "v"(xh));
          tg[e] = p == 0 ? gr[e] * xh : __builtin_fmaf(gr[e], xh, tg[e]);
          if (p == 0) tb[e] = gr[e];
          else asm volatile("v_add_f32 %0, %0, %1" : "+v"(tb[e]) : "v"(gr[e]));
        }
        __builtin_amdgcn_sched_barrier(0);             // interleaved passes would keep their unpacked values live together
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(cgs[4 * d + e]) : "v"(sg), "v"(tg[e]));
        asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(cbs[4 * d + e]) : "v"(sg), "v"(tb[e]));
      }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      m1[p] = wave_group_sum<7>(m1[p] * sg);
      m2[p] = wave_group_sum<7>(m2[p] * sg);
      if (t.ch == 0) *reinterpret_cast<float2*>(s_row + ((parity * t.nstrips + t.wave) * 32 + t.rsub + 8 * p) * 2) = make_float2(m1[p], m2[p]);
    }
    lds_barrier();
    if (AHEAD) wait_all_loads();                         // before the store, see jf_layernorm_rows.hpp
    // lanes 2 i and 2 i + 1: the two means of row i, the strips in a fixed order (the share of this workgroup's column range; the
    // second kernel adds the ranges)
    if (threadIdx.x < 64)
      row_means[2 * ((int64_t)blockIdx.y * rows + bi * 32) + threadIdx.x] =
          sum_over_strips(s_row + parity * t.nstrips * 64 + threadIdx.x, t.nstrips) * inv_cols;
  }

  float sums[8];
  reduce_rows32(cgs, cbs, sums);
  if (t.ok && (t.rsub & 1) == 0)
    store_partials(partials + (int64_t)blockIdx.x * 2 * cols + t.col - 16 * t.ch + reduced_column(threadIdx.x & 63), cols, sums);
}

// Column sums: the partial rows of dgamma | dbeta (2 cols wide) of one group of 64 columns, added in a fixed order by a
// workgroup of NW waves: wave w takes rows w, w + NW, ... in eight independent chains, which keep loads in flight, and wave 0
// adds the NW results in wave order.  The two-kernel backward does this in workgroups in front of its second kernel's own,
// which need nothing of it, so that it costs no launch (3200 x 896 at block 128: 22.4 -> 19.4 us forward and backward).
template <int NW>
__device__ __forceinline__ void colsum_group(int group, const float* __restrict__ partials, int nparts, int cols2,
                                             float* __restrict__ dgamma, float* __restrict__ dbeta) {
  __shared__ float s_part[NW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = group * 64 + lane;
  float acc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  if (c < cols2) {
    int p = wave;
    // sixteen rows requested together, all that a wave has of 256 partial rows
    for (; p + 15 * NW < nparts; p += 16 * NW) {
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = partials[(int64_t)(p + NW * j) * cols2 + c];
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j & 7] += v[j];
    }
    for (; p + 7 * NW < nparts; p += 8 * NW) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = partials[(int64_t)(p + NW * j) * cols2 + c];
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += v[j];
    }
    for (; p < nparts; p += NW) acc[0] += partials[(int64_t)p * cols2 + c];
  }
  s_part[wave][lane] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  __syncthreads();
  if (wave == 0 && c < cols2) {
    double v = 0.0;   // (sixteen roundings fewer; nothing to add to the time)
#pragma unroll
    for (int w = 0; w < NW; ++w) v += (double)s_part[w][lane];
    const int half = cols2 / 2;
    if (c < half) dgamma[c] = (float)v;
    else dbeta[c - half] = (float)v;
  }
}
// the same as a launch of its own, behind the one-pass backward
__global__ void __launch_bounds__(1024) colsum_kernel(const float* __restrict__ partials, int nparts, int cols2,
                                                       float* __restrict__ dgamma, float* __restrict__ dbeta) {
  colsum_group<16>(blockIdx.x, partials, nparts, cols2, dgamma, dbeta);
}
// what the second kernel of the two-kernel backward needs for it; groups = 0: nothing
struct ColumnSums {
  const float* partials;
  float *dgamma, *dbeta;
  int nparts, groups;
};

// Second kernel: dx on 32 x 128 strips, one wave each, from the row means q1 = mean_C(ghat), q2 = mean_C(ghat xhat)
// that the first kernel left (one share per range of 2048 columns): dx = ug a_c + ux b + d with per-row
// b = -rstd q2 sx rstd and d, and per-column a_c = rstd sg gamma_c (u = code + 128), then Eq. 1.  Rows may be of any
// width.
template <StorePolicy SP>
__global__ void __launch_bounds__(64 * kStripWaves) layernorm_bwd_apply_strip32_kernel(
    const int8_t* __restrict__ G, const int8_t* __restrict__ X, const float* __restrict__ SG, const float* __restrict__ SX, int rows, int cols, int groups,
    int ranges, const float* __restrict__ gamma, const float* __restrict__ mean_in, const float* __restrict__ rstd_in, const float* __restrict__ row_means,
    int8_t* __restrict__ dX, float* __restrict__ SdX, const ColumnSums cs) {
  if ((int)blockIdx.x < groups) {
    colsum_group<kStripWaves>(blockIdx.x, cs.partials, cs.nparts, 2 * cols, cs.dgamma, cs.dbeta);
    return;
  }
  const Strip32 t(rows, cols, groups);
  if (!t.inside) return;   // a whole wave; the strip kernels have no workgroup barrier
  const int64_t pass = (int64_t)8 * cols;
  uint4 px[4], pg[4];
  float mu[4], rs[4];
  float2 q[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    px[p] = *reinterpret_cast<const uint4*>(X + t.base + p * pass);
    pg[p] = *reinterpret_cast<const uint4*>(G + t.base + p * pass);
    const int row = t.bi * 32 + t.rsub + 8 * p;
    mu[p] = mean_in[row];
    rs[p] = rstd_in[row];
    q[p] = *reinterpret_cast<const float2*>(row_means + 2 * (int64_t)row);
    for (int cr = 1; cr < ranges; ++cr) {   // rows wider than 2048 columns: the column ranges in a fixed order
      const float2 part = *reinterpret_cast<const float2*>(row_means + 2 * ((int64_t)cr * rows + row));
      q[p].x += part.x;
      q[p].y += part.y;
    }
  }
  const float sx = SX[t.block_index()], sg = SG[t.block_index()];
  float gm[16];
  load16f(gamma + (t.ok ? t.col : t.c0), gm);
  float y[4][16];
  float m = 0.0f;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    float ux[16], ug[16];
    unpack16_biased(px[p], ux);
    unpack16_biased(pg[p], ug);
    const float kx = sx * rs[p], cx0 = __builtin_fmaf(-128.0f, kx, -mu[p] * rs[p]);
    const float kxm = -rs[p] * q[p].y * kx, krow = -rs[p] * __builtin_fmaf(cx0, q[p].y, q[p].x);
    const float rsg = rs[p] * sg;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float a = rsg * gm[e];
      const float k = __builtin_fmaf(a, -128.0f, krow);
      y[p][e] = __builtin_fmaf(ux[e], kxm, __builtin_fmaf(ug[e], a, k));
    }
    m = amax16(m, y[p]);
  }
  float scale;
  double inv;
  strip32_block_scale(m, scale, inv);
  if (!t.ok) return;
  if ((t.lane & 57) == 0) store_scale<SP>(&SdX[t.block_index()], scale);
#pragma unroll
  for (int p = 0; p < 4; ++p) store_as<SP>(dX + t.base + p * pass, quantize16(y[p], inv));
}

// Row statistics of LayerNorm from the row partials that the preceding Add wrote (App. A, LayerNorm paragraph):
//   mean_i = (1 / L_C) sum_j row_mean[j][i],  var_i = max((1 / C) sum_j row_sumsq[j][i] - mean_i^2, 0),
// summed in double in a fixed order; rstd as the hardware reciprocal square root plus one Newton step.  The partials are
// stored block-column-major ((C / B) x N): a workgroup owns 64 consecutive rows, lane = row, so every load of a wave is
// 64 consecutive floats; its waves (4 to 16, about one per four block columns) take the block columns j = w, w + waves,
// ... and their shares are added through LDS in wave order.
__global__ void __launch_bounds__(1024) row_stats_from_partials_kernel(const float* __restrict__ row_mean,
                                                                        const float* __restrict__ row_sumsq, float eps,
                                                                        int rows, int lc, int cols, int NW,
                                                                        float* __restrict__ mean_out, float* __restrict__ rstd_out) {
  __shared__ double s_part[2][16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = min((int)blockIdx.x * 64 + lane, rows - 1);   // lanes past the last row repeat it and write nothing
  double s = 0.0, q = 0.0;
  for (int j0 = wave; j0 < lc; j0 += 4 * NW) {   // four block columns in flight at a time
    float m[4], v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t at = (int64_t)min(j0 + k * NW, lc - 1) * rows + row;
      m[k] = row_mean[at];
      v[k] = row_sumsq[at];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s += j0 + k * NW < lc ? (double)m[k] : 0.0;
      q += j0 + k * NW < lc ? (double)v[k] : 0.0;
    }
  }
  s_part[0][wave][lane] = s;
  s_part[1][wave][lane] = q;
  __syncthreads();
  if (wave != 0 || (int)blockIdx.x * 64 + lane >= rows) return;
  s = sum_over_strips(&s_part[0][0][lane], NW);
  q = sum_over_strips(&s_part[1][0][lane], NW);
  const double mu = s / (double)lc;
  const float var = fmaxf((float)(q / (double)cols - mu * mu), 0.0f);
  const float ve = var + eps;
  float rs = __builtin_amdgcn_rsqf(ve);
  rs = rs * __builtin_fmaf(-0.5f * ve * rs, rs, 1.5f);
  mean_out[row] = (float)mu;
  rstd_out[row] = rs;
}

// LayerNorm at block size 32 from given row statistics (App. A: the operator is handed the row mean and rstd):
// y = (x - mean) rstd gamma + beta on 32 x 128 strips, one wave each, like the other element-wise operators --
// no workgroup needs a whole row, so rows may be of any width.
template <StorePolicy SP>
__global__ void __launch_bounds__(64 * kStripWaves) layernorm_apply_strip32_kernel(const int8_t* __restrict__ X, const float* __restrict__ SX,
                                                                     const float* __restrict__ gamma, const float* __restrict__ beta,
                                                                     const float* __restrict__ mean_in, const float* __restrict__ rstd_in,
                                                                     int rows, int cols, int8_t* __restrict__ Y, float* __restrict__ SY) {
  const Strip32 t(rows, cols);
  if (!t.inside) return;   // a whole wave; the strip kernels have no workgroup barrier
  const int64_t pass = (int64_t)8 * cols;
  uint4 px[4];
  float mu[4], rs[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    px[p] = *reinterpret_cast<const uint4*>(X + t.base + p * pass);
    mu[p] = mean_in[t.bi * 32 + t.rsub + 8 * p];
    rs[p] = rstd_in[t.bi * 32 + t.rsub + 8 * p];
  }
  const float sx = SX[t.block_index()];
  float gm[16], bt[16];
  const int gcol = t.ok ? t.col : t.c0;
  load16f(gamma + gcol, gm);
  load16f(beta + gcol, bt);
  float y[4][16];
  float m = 0.0f;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    float u[16];
    unpack16_biased(px[p], u);
    const float k1 = sx * rs[p], kb = __builtin_fmaf(-128.0f, k1, -mu[p] * rs[p]);
#pragma unroll
    for (int e = 0; e < 16; ++e) y[p][e] = __builtin_fmaf(__builtin_fmaf(u[e], k1, kb), gm[e], bt[e]);
    m = amax16(m, y[p]);
  }
  float scale;
  double inv;
  strip32_block_scale(m, scale, inv);
  if (!t.ok) return;
  if ((t.lane & 57) == 0) store_scale<SP>(&SY[t.block_index()], scale);
#pragma unroll
  for (int p = 0; p < 4; ++p) store_as<SP>(Y + t.base + p * pass, quantize16(y[p], inv));
}

// The same two element-wise operators at block sizes 64 and 128: one workgroup of four waves owns B rows x 128 columns
// (two blocks resp. one); wave w owns rows [w B/4, (w+1) B/4) in B/32 passes of 8 rows with the lane mapping of the
// strips (lane = (row l / 8, 16-byte chunk l % 8): full 128-byte lines); the block max-abs goes over the lanes of a
// block column inside a wave and over the four waves through LDS.  MODE 0: y = (x - mean) rstd gamma + beta (forward),
// MODE 1: dx from the row means of the sums kernel (backward).
template <int B, int MODE, StorePolicy SP>
__global__ void __launch_bounds__(256) layernorm_tile_kernel(const int8_t* __restrict__ G, const int8_t* __restrict__ X, const float* __restrict__ SG,
                                                              const float* __restrict__ SX, int rows, int cols, int groups, int ranges,
                                                              const float* __restrict__ gamma, const float* __restrict__ beta,
                                                              const float* __restrict__ mean_in, const float* __restrict__ rstd_in,
                                                              const float* __restrict__ row_means, int8_t* __restrict__ Y,
                                                              float* __restrict__ SY, const ColumnSums cs) {
  constexpr int P = B / 32;
  __shared__ float s_amax[4][4];
  if constexpr (MODE == 1) {
    if ((int)blockIdx.x < groups) {
      colsum_group<4>(blockIdx.x, cs.partials, cs.nparts, 2 * cols, cs.dgamma, cs.dbeta);
      return;
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ch = lane & 7, rsub = lane >> 3;
  const TileIndex wg = tile_of_workgroup((cols + 127) / 128, MODE == 1 ? groups : 0);
  const int col = wg.x * 128 + 16 * ch;
  const int r0 = wg.y * B + wave * (B / 4);
  const bool col_ok = col < cols;
  const int lc = cols / B, bi = wg.y;

  float y[P][16];
  float m = 0.0f;
  if (col_ok) {
    const float sx = SX[(int64_t)bi * lc + col / B];
    float gm[16], bt[16];
    load16f(gamma + col, gm);
    float sg = 0.0f;
    if (MODE == 0) load16f(beta + col, bt);
    else sg = SG[(int64_t)bi * lc + col / B];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int row = r0 + 8 * p + rsub;
      const float mu = mean_in[row], rs = rstd_in[row];
      float ux[16];
      unpack16_biased(*reinterpret_cast<const uint4*>(X + (int64_t)row * cols + col), ux);
      const float kx = sx * rs, cx0 = __builtin_fmaf(-128.0f, kx, -mu * rs);   // xhat = ux kx + cx0, ux = code + 128
      if (MODE == 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) y[p][e] = __builtin_fmaf(__builtin_fmaf(ux[e], kx, cx0), gm[e], bt[e]);
      } else {
        float2 q = *reinterpret_cast<const float2*>(row_means + 2 * (int64_t)row);
        for (int cr = 1; cr < ranges; ++cr) {   // rows wider than 2048 columns: the column ranges in a fixed order
          const float2 part = *reinterpret_cast<const float2*>(row_means + 2 * ((int64_t)cr * rows + row));
          q.x += part.x;
          q.y += part.y;
        }
        float ug[16];
        unpack16_biased(*reinterpret_cast<const uint4*>(G + (int64_t)row * cols + col), ug);
        const float kxm = -rs * q.y * kx, krow = -rs * __builtin_fmaf(cx0, q.y, q.x), rsg = rs * sg;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float a = rsg * gm[e];
          y[p][e] = __builtin_fmaf(ux[e], kxm, __builtin_fmaf(ug[e], a, __builtin_fmaf(a, -128.0f, krow)));
        }
      }
      m = amax16(m, y[p]);
    }
  }
  m = wave_group_max<56 | (B / 16 - 1)>(m);
  // s_amax[wave][32-column group]; the in-wave reduction already covered the whole block width
  if ((lane & 57) == 0) s_amax[wave][ch >> 1] = m;
  __syncthreads();
  m = fmaxf(fmaxf(s_amax[0][ch >> 1], s_amax[1][ch >> 1]), fmaxf(s_amax[2][ch >> 1], s_amax[3][ch >> 1]));
  float scale;
  double inv;
  block_scale(m, scale, inv);
  if (!col_ok) return;
  if (wave == 0 && rsub == 0 && (col % B) == 0) store_scale<SP>(&SY[(int64_t)bi * lc + col / B], scale);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int row = r0 + 8 * p + rsub;
    store_as<SP>(Y + (int64_t)row * cols + col, quantize16(y[p], inv));
  }
}

// ------------------------------------------------------------------------------------------------ host
}  // namespace jf

// Strips are shared evenly by the column ranges.  The next row block is requested ahead (AHEAD) where a workgroup takes four or more:
// 131072 x 1088 at block 64, whole backward pass, 175 -> 165 us, 262144 x 3072 850 -> 815; with one or two the way through LDS costs
// more than it hides (4096 x 4096 22.0 and 23.1, 32768 x 2048 69.2 and 70.4).
static void launch_ln_bwd_sums(const int8_t* dY, const float* SdY, const int8_t* X, const float* SX, const float* gamma, const float* mean, const float* rstd,
                               int64_t N, int64_t C, int32_t block, float* row_means, float* partials, dim3 grid, hipStream_t st) {
  using namespace jf;
  const int ns = (int)(((C + 127) / 128 + grid.y - 1) / grid.y);   // waves
  const auto launch = [&](auto kernel, int wave_bytes) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * ns), ns * wave_bytes, st, dY, X, SdY, SX, (int)N, (int)C, block_log2(block), ns, gamma, mean, rstd,
                       row_means, partials);
  };
  if (N / 32 < 4 * (int64_t)grid.x) return launch(layernorm_bwd_sums_kernel<false>, kSumsRowBytes);
  constexpr int BYTES = kSumsRowBytes + kSumsWaveBytes;
  static_assert(16 * BYTES <= 160 * 1024, "sixteen waves share the LDS of a compute unit");
  // (see launch_rows)
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(layernorm_bwd_sums_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, 16 * BYTES) != hipSuccess) return;
  launch(layernorm_bwd_sums_kernel<true>, BYTES);
}

// A statistics kernel (from the Add's partials, or from the codes), then the normalisation on tiles.
static int32_t layernorm_fwd(const int8_t* X, const float* SX, const float* row_mean, const float* row_sumsq,
                             const float* gamma, const float* beta, float eps, int64_t N, int64_t C, int32_t block,
                             int8_t* Y, float* SY, float* mean, float* rstd, void* stream) {
  using namespace jf;
  int32_t rc = check_eltwise(X, SX, Y, SY, N, C, block);
  if (rc != JF_OK) return rc;
  if (!gamma || !beta || !mean || !rstd) return JF_ERR_NULL;
  if (!aligned16(gamma) || !aligned16(beta) || !aligned4(mean) || !aligned4(rstd)) return JF_ERR_ALIGN;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const bool whole_rows = layernorm_rows_fits(N, C, block, false);
  if (whole_rows || (row_mean == nullptr && layernorm_wide_fits(N, C, block, false))) {   // one pass over the operands
    LayerNormRows a{};
    a.X = X; a.SX = SX; a.row_mean = row_mean; a.row_sumsq = row_sumsq; a.gamma = gamma; a.beta = beta; a.eps = eps;
    a.rows = (int)N; a.cols = (int)C; a.Y = Y; a.SY = SY; a.mean = mean; a.rstd = rstd;
    const int64_t grid_bytes = N / block * (C / block) * 4, part_bytes = N * (C / block) * 4;
    const MemRange in[] = {{X, N * C}, {SX, grid_bytes}, {row_mean, part_bytes}, {row_sumsq, part_bytes}, {gamma, 4 * C}, {beta, 4 * C}};
    const MemRange out[] = {{Y, N * C}, {SY, grid_bytes}, {mean, 4 * N}, {rstd, 4 * N}};
    if (!whole_rows) launch_layernorm_wide(a, st);
    else if (block == 32 && layernorm_split_parts(N, C, false) > 1 && !any_overlap(out, in)) launch_layernorm_split(a, st);
    else (block == 32 ? launch_layernorm_rows_b32 : block == 64 ? launch_layernorm_rows_b64 : launch_layernorm_rows_b128)(a, st);
    return launch_status();
  }
  if (row_mean != nullptr) {
    const int waves = (int)std::min<int64_t>(16, std::max<int64_t>(4, C / block / 4));
    hipLaunchKernelGGL(row_stats_from_partials_kernel, dim3((unsigned)((N + 63) / 64)), dim3(64 * waves), 0, st, row_mean, row_sumsq,
                       eps, (int)N, (int)(C / block), (int)C, waves, mean, rstd);
  } else {
    const int waves = (int)std::min<int64_t>(16, (C + 127) / 128);
    hipLaunchKernelGGL(layernorm_row_stats_kernel, dim3((unsigned)(N / 32)), dim3(64 * waves), 0, st, X, SX, eps, (int)N, (int)C,
                       block_log2(block), waves, mean, rstd);
  }
  rc = launch_status();
  if (rc != JF_OK) return rc;
  const dim3 tiles(tile_grid((C + 127) / 128, N / block));
  const float* none = nullptr;
  with_store_policy(N, C, [&](auto sp) {
    constexpr StorePolicy SP = decltype(sp)::value;
    if (block == 32)
      hipLaunchKernelGGL((layernorm_apply_strip32_kernel<SP>), strip_grid(N, C), dim3(64 * kStripWaves), 0, st, X, SX, gamma, beta, mean,
                         rstd, (int)N, (int)C, Y, SY);
    else if (block == 64)
      hipLaunchKernelGGL((layernorm_tile_kernel<64, 0, SP>), tiles, dim3(256), 0, st, (const int8_t*)nullptr, X, none, SX, (int)N, (int)C, 0, 1, gamma,
                         beta, (const float*)mean, (const float*)rstd, none, Y, SY, ColumnSums{});
    else
      hipLaunchKernelGGL((layernorm_tile_kernel<128, 0, SP>), tiles, dim3(256), 0, st, (const int8_t*)nullptr, X, none, SX, (int)N, (int)C, 0, 1, gamma,
                         beta, (const float*)mean, (const float*)rstd, none, Y, SY, ColumnSums{});
  });
  return launch_status();
}

extern "C" int32_t jf_layernorm_q(const int8_t* X, const float* SX, const float* gamma, const float* beta, float eps,
                                  int64_t N, int64_t C, int32_t block, int8_t* Y, float* SY, float* mean, float* rstd,
                                  void* stream) {
  return layernorm_fwd(X, SX, nullptr, nullptr, gamma, beta, eps, N, C, block, Y, SY, mean, rstd, stream);
}

extern "C" int32_t jf_layernorm_q_partials(const int8_t* X, const float* SX, const float* row_mean,
                                           const float* row_sumsq, const float* gamma, const float* beta, float eps,
                                           int64_t N, int64_t C, int32_t block, int8_t* Y, float* SY, float* mean,
                                           float* rstd, void* stream) {
  if (!row_mean || !row_sumsq) return JF_ERR_NULL;
  if (!jf::aligned4(row_mean) || !jf::aligned4(row_sumsq)) return JF_ERR_ALIGN;
  return layernorm_fwd(X, SX, row_mean, row_sumsq, gamma, beta, eps, N, C, block, Y, SY, mean, rstd, stream);
}

// LayerNorm backward behind both entry points: `partials` is the caller's workspace or this library's static
// scratch; every argument has been validated.
static int32_t layernorm_bwd_launch(const int8_t* dY, const float* SdY, const int8_t* X, const float* SX,
                                    const float* gamma, const float* mean, const float* rstd, int64_t N, int64_t C,
                                    int32_t block, int8_t* dX, float* SdX, float* dgamma, float* dbeta, float* partials,
                                    hipStream_t st) {
  using namespace jf;
  int nparts = (int)ln_bwd_partial_rows(N);
  // In place (dX over dY or X, dgamma over gamma) the column sums are taken in a kernel behind the one that writes dX:
  // where they come from workgroups beside it, those read what dX replaces, or replace what dX is formed from.
  const int64_t grid_bytes = N / block * (C / block) * 4;
  const MemRange in[] = {{dY, N * C}, {SdY, grid_bytes}, {X, N * C}, {SX, grid_bytes}, {gamma, 4 * C}, {mean, 4 * N}, {rstd, 4 * N}};
  const MemRange out[] = {{dX, N * C}, {SdX, grid_bytes}}, sums[] = {{dgamma, 4 * C}, {dbeta, 4 * C}};
  const bool sums_in_place = any_overlap(sums, in);
  const auto launch_colsum = [&]() {
    hipLaunchKernelGGL(colsum_kernel, dim3((unsigned)((2 * C + 63) / 64)), dim3(1024), 0, st, partials, nparts, (int)(2 * C), dgamma, dbeta);
    return launch_status();
  };
  const bool whole_rows = layernorm_rows_fits(N, C, block, true);
  if (whole_rows || layernorm_wide_fits(N, C, block, true)) {   // one pass over the operands
    LayerNormBwdRows a{};
    a.G = dY; a.SG = SdY; a.X = X; a.SX = SX; a.gamma = gamma; a.mean = mean; a.rstd = rstd; a.rows = (int)N; a.cols = (int)C;
    a.dX = dX; a.SdX = SdX; a.partials = partials;
    a.dgamma = dgamma; a.dbeta = dbeta;
    if (!whole_rows) nparts = launch_layernorm_bwd_wide(a, st);
    else if (block == 32 && layernorm_split_parts(N, C, true) > 1 && !sums_in_place && !any_overlap(out, in)) nparts = launch_layernorm_bwd_split(a, st);
    else
      nparts = (block == 32 ? launch_layernorm_bwd_rows_b32 : block == 64 ? launch_layernorm_bwd_rows_b64 : launch_layernorm_bwd_rows_b128)(
          a, sums_in_place || any_overlap(out, in), st);
    const int32_t rc = launch_status();
    return rc != JF_OK || nparts == 0 ? rc : launch_colsum();
  }
  // the workspace holds the partial rows, then the two row means of every row (per range of 2048 columns)
  float* row_means = partials + (size_t)nparts * 2 * (size_t)C;
  const int ranges = (int)((C + 2047) / 2048);
  launch_ln_bwd_sums(dY, SdY, X, SX, gamma, mean, rstd, N, C, block, row_means, partials, dim3((unsigned)nparts, (unsigned)ranges), st);
  const int32_t rc1 = launch_status();
  if (rc1 != JF_OK) return rc1;
  const ColumnSums cs = {partials, dgamma, dbeta, nparts, sums_in_place ? 0 : (int)((2 * C + 63) / 64)};
  const dim3 tiles(cs.groups + tile_grid((C + 127) / 128, N / block)), strips(cs.groups + strip_grid(N, C).x);
  const float* none = nullptr;
  with_store_policy(N, C, [&](auto sp) {
    constexpr StorePolicy SP = decltype(sp)::value;
    if (block == 32)
      hipLaunchKernelGGL((layernorm_bwd_apply_strip32_kernel<SP>), strips, dim3(64 * kStripWaves), 0, st, dY, X, SdY, SX, (int)N, (int)C, cs.groups,
                         ranges, gamma, mean, rstd, row_means, dX, SdX, cs);
    else if (block == 64)
      hipLaunchKernelGGL((layernorm_tile_kernel<64, 1, SP>), tiles, dim3(256), 0, st, dY, X, SdY, SX, (int)N, (int)C, cs.groups, ranges, gamma, none,
                         mean, rstd, (const float*)row_means, dX, SdX, cs);
    else
      hipLaunchKernelGGL((layernorm_tile_kernel<128, 1, SP>), tiles, dim3(256), 0, st, dY, X, SdY, SX, (int)N, (int)C, cs.groups, ranges, gamma, none,
                         mean, rstd, (const float*)row_means, dX, SdX, cs);
  });
  const int32_t rc2 = launch_status();
  return rc2 != JF_OK || !sums_in_place ? rc2 : launch_colsum();
}

static int32_t layernorm_bwd_check(const int8_t* dY, const float* SdY, const int8_t* X, const float* SX,
                                   const float* gamma, const float* mean, const float* rstd, int64_t N, int64_t C,
                                   int32_t block, int8_t* dX, float* SdX, float* dgamma, float* dbeta) {
  using namespace jf;
  int32_t rc = check_eltwise(X, SX, dX, SdX, N, C, block);
  if (rc != JF_OK) return rc;
  if (!dY || !SdY || !gamma || !mean || !rstd || !dgamma || !dbeta) return JF_ERR_NULL;
  if (!aligned16(dY) || !aligned4(SdY) || !aligned16(gamma) || !aligned4(mean) || !aligned4(rstd) ||
      !aligned4(dgamma) || !aligned4(dbeta))
    return JF_ERR_ALIGN;
  return JF_OK;
}

extern "C" int32_t jf_layernorm_q_bwd(const int8_t* dY, const float* SdY, const int8_t* X, const float* SX,
                                      const float* gamma, const float* mean, const float* rstd, int64_t N, int64_t C,
                                      int32_t block, int8_t* dX, float* SdX, float* dgamma, float* dbeta, void* ws,
                                      size_t ws_bytes, void* stream) {
  int32_t rc = layernorm_bwd_check(dY, SdY, X, SX, gamma, mean, rstd, N, C, block, dX, SdX, dgamma, dbeta);
  if (rc != JF_OK) return rc;
  const size_t need = jf_workspace_bytes(JF_OP_LAYERNORM_BWD, N, C, 0, block);
  if (!ws || ws_bytes < need) return JF_ERR_WORKSPACE;
  if (!jf::aligned16(ws)) return JF_ERR_ALIGN;
  return layernorm_bwd_launch(dY, SdY, X, SX, gamma, mean, rstd, N, C, block, dX, SdX, dgamma, dbeta,
                              static_cast<float*>(ws), reinterpret_cast<hipStream_t>(stream));
}

// ------------------------------------------------------------------------------------------------
// The entry point that allocates nothing: jf_layernorm_q_bwd with its workspace (the partial rows of
// dgamma | dbeta) in a static device array instead of a caller-provided buffer.  In host code the array's
// name is only a handle: its device address is looked up once per device, with that device current, and that
// pointer is what the kernels receive.  Every GPU holds its own copy of the array until the process ends.
static __device__ __align__(256) unsigned char scratch[JF_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, once looked up

// Device address of the static scratch on the current device (nullptr and *rc = JF_ERR_LAUNCH on failure).
void* static_scratch(int32_t* rc) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices)) e = hipErrorInvalidDevice;
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e == hipSuccess && p == nullptr) e = hipErrorInvalidSymbol;
      if (e == hipSuccess) g_scratch_ptr[dev] = p;
    }
    if (e == hipSuccess) return g_scratch_ptr[dev];
  }
  jf::g_last_hip_error = (int32_t)e;
  *rc = JF_ERR_LAUNCH;
  return nullptr;
}
}  // namespace

extern "C" int32_t jf_layernorm_q_bwd_static(const int8_t* dY, const float* SdY, const int8_t* X, const float* SX,
                                             const float* gamma, const float* mean, const float* rstd, int64_t N,
                                             int64_t C, int32_t block, int8_t* dX, float* SdX, float* dgamma,
                                             float* dbeta, void* stream) {
  int32_t rc = layernorm_bwd_check(dY, SdY, X, SX, gamma, mean, rstd, N, C, block, dX, SdX, dgamma, dbeta);
  if (rc != JF_OK) return rc;
  if (jf_workspace_bytes(JF_OP_LAYERNORM_BWD, N, C, 0, block) > (size_t)JF_STATIC_SCRATCH_BYTES) return JF_ERR_WORKSPACE;
  void* const ptr = static_scratch(&rc);
  if (ptr == nullptr) return rc;
  // Nothing in the scratch has to start at zero: every partial row that the second kernel reads is written
  // in full by the first one of the same call.
  return layernorm_bwd_launch(dY, SdY, X, SX, gamma, mean, rstd, N, C, block, dX, SdX, dgamma, dbeta,
                              static_cast<float*>(ptr), reinterpret_cast<hipStream_t>(stream));
}
