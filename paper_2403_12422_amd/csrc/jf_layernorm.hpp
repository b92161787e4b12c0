// What the LayerNorm sources share: jf_layernorm.hip (entry points; sums kernels + operators on tiles), jf_layernorm_rows.hpp (one
// pass over whole rows) and jf_layernorm_wide.hip (the same for wider rows).
#pragma once
#include "jf_rowops.hpp"

namespace jf {

// s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8
__device__ __forceinline__ void wait_all_loads() {
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));
  asm volatile("" ::: "memory");
}
// LDS writes of all waves before, LDS reads after; global loads stay in flight (unlike __syncthreads)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));
  asm volatile("s_barrier" ::: "memory");
}
// a wave's own LDS writes before its own reads
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// exact sums of the 16 codes of a chunk and of their squares
__device__ __forceinline__ void chunk_moments(const uint4& p, int& s1, int& s2) {
  s1 = __builtin_amdgcn_sdot4((int)p.x, 0x01010101, 0, false);
  s1 = __builtin_amdgcn_sdot4((int)p.y, 0x01010101, s1, false);
  s1 = __builtin_amdgcn_sdot4((int)p.z, 0x01010101, s1, false);
  s1 = __builtin_amdgcn_sdot4((int)p.w, 0x01010101, s1, false);
  s2 = __builtin_amdgcn_sdot4((int)p.x, (int)p.x, 0, false);
  s2 = __builtin_amdgcn_sdot4((int)p.y, (int)p.y, s2, false);
  s2 = __builtin_amdgcn_sdot4((int)p.z, (int)p.z, s2, false);
  s2 = __builtin_amdgcn_sdot4((int)p.w, (int)p.w, s2, false);
}

// Signed codes of one packed dword as floats (a byte-select conversion each).
__device__ __forceinline__ void unpack4(uint32_t w, float (&c)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = (float)(int)(int8_t)(w >> (8 * k));
}
__device__ __forceinline__ uint32_t dword_of(const uint4& v, int d) { return d == 0 ? v.x : (d == 1 ? v.y : (d == 2 ? v.z : v.w)); }

// v[0] + v[64] + v[128] + ... of the `strips` waves of a team, in that order, four LDS reads in flight at a time (one after
// the other they are one LDS latency per strip, beside which nothing runs where a workgroup has a single row group).
template <class T>
__device__ __forceinline__ T sum_over_strips(const T* v, int strips) {
  T sum = 0;
  for (int w = 0; w < strips; w += 4) {
    T q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = v[64 * min(w + j, strips - 1)];
#pragma unroll
    for (int j = 0; j < 4; ++j) sum += w + j < strips ? q[j] : (T)0;
  }
  return sum;
}

// Sums over the 8 row lanes of a wave (lane bits 3, 4, 5, in that order) of 16 + 16 values.  The half-row swaps of two values
// and one addition reduce both: 80 instructions where 32 butterflies take 320, at the end of a workgroup with nothing beside it
// (with two rows of ghat kept: 8192 x 1280 17.2 -> 15.0 us, 4096 x 768 11.5 -> 10.1, 1056 x 800 7.1 -> 6.5).  Lane (bits 4, 5) ends with
// values 4 (bit 4 + 2 (bit 5)) + j of a (out[j]) and of b (out[4 + j]), j = 0 .. 3, which lie beside each other in memory.
__device__ __forceinline__ void reduce_rows32(const float (&a)[16], const float (&b)[16], float (&out)[8]) {
  const auto half = [](float x, float y, auto swap) __attribute__((always_inline)) {
    const auto p = swap(__builtin_bit_cast(int, x), __builtin_bit_cast(int, y));
    return __builtin_bit_cast(float, (int)p[0]) + __builtin_bit_cast(float, (int)p[1]);
  };
  const auto swap16 = [](int x, int y) { return __builtin_amdgcn_permlane16_swap(x, y, false, false); };
  const auto swap32 = [](int x, int y) { return __builtin_amdgcn_permlane32_swap(x, y, false, false); };
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = wave_group_sum<8>(j < 4 ? a[4 * k + j] : b[4 * k + j - 4]);
    out[j] = half(half(v[0], v[1], swap16), half(v[2], v[3], swap16), swap32);
  }
}
// First of the four columns of the strip whose sums a lane ends with.
__device__ __forceinline__ int reduced_column(int lane) { return 16 * (lane & 7) + 4 * (((lane >> 4) & 1) | ((lane >> 5) << 1)); }
// A strip's part of a partial row of dgamma | dbeta: 512 bytes of each in two instructions, whole lines, so they can be written through like
// other results (in pieces of a float, left for the end of the kernel to write back, and the sums of them by eights, 8192 x 1280 14.6 us; so 14.1).
__device__ __forceinline__ void store_partials(float* dgamma, int cols, const float (&sums)[8]) {
  store_out(dgamma, v4f{sums[0], sums[1], sums[2], sums[3]});
  store_out(dgamma + cols, v4f{sums[4], sums[5], sums[6], sums[7]});
}

// Sums over the 32 lanes of each half wave of 32 values, by halves: a step adds two values at once, lanes with the bit clear for one,
// with it set for the other (rows of lanes, then halves of a row and of those, by masked moves; then whole quads): 110 instructions, a
// butterfly for each value takes 480.  Every lane ends with one of the 32 sums in v[0]; returned is which.
__device__ __forceinline__ int reduce_rows_of_32(float (&v)[32], int lane) {
  const auto bits = [](float x) __attribute__((always_inline)) { return __builtin_bit_cast(int, x); };
  const auto real = [](int x) __attribute__((always_inline)) { return __builtin_bit_cast(float, x); };
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const auto p = __builtin_amdgcn_permlane16_swap(bits(v[2 * j]), bits(v[2 * j + 1]), false, false);
    v[j] = real((int)p[0]) + real((int)p[1]);
  }
  // of a and b, lanes in BANKS take b, each plus its partner's across STEP
#define JF_MERGE(A, B, BANKS, STEP)                                                                        \
  (real(__builtin_amdgcn_update_dpp(bits(A), bits(B), 0xE4, 0xf, BANKS, false)) +                          \
   real(__builtin_amdgcn_mov_dpp(__builtin_amdgcn_update_dpp(bits(B), bits(A), 0xE4, 0xf, BANKS, false), STEP, 0xf, 0xf, false)))
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = JF_MERGE(v[2 * j], v[2 * j + 1], 0xC, 0x128);    // across 8 lanes
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = JF_MERGE(v[2 * j], v[2 * j + 1], 0xA, 0x141);    // lane i and 7 - i
#undef JF_MERGE
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] += lane_xor_f32<0>(v[j]);
    v[j] += lane_xor_f32<1>(v[j]);
  }
  const int j = lane & 3;
  v[0] = j == 0 ? v[0] : j == 1 ? v[1] : j == 2 ? v[2] : v[3];
  return 8 * j + (lane & 4) + ((lane >> 2) & 2) + ((lane >> 4) & 1);
}

struct LayerNormRows {
  const int8_t* X;
  const float *SX, *row_mean, *row_sumsq, *gamma, *beta;   // row partials nullable: statistics of the codes themselves
  float eps;
  int rows, cols;
  int8_t* Y;
  float *SY, *mean, *rstd;
  int strips, teams;              // set by the launcher, like the reciprocals
  double inv_cols, inv_blocks;
};
struct LayerNormBwdRows {
  const int8_t* G;
  const float* SG;
  const int8_t* X;
  const float *SX, *gamma, *mean, *rstd;
  int rows, cols;
  int8_t* dX;
  float *SdX, *partials, *dgamma, *dbeta;
  int strips, teams, row_wgs;     // row_wgs: workgroups that own rows; those behind them own columns
  float inv_cols;
};

// Arguments of the kernels whose workgroups own whole rows: what their first loads need in the dwords that are preloaded, the rest read
// behind those.  layout: strips, teams and waves of a workgroup, 8 bits each; wgs: workgroups that own rows.
struct LayerNormRowsArgs {
  const int8_t* X;
  const float *SX, *first, *second;   // row partials if there are any, else gamma and beta
  int rows, cols, layout, wgs;
  LayerNormRows all;
};
struct LayerNormBwdRowsArgs {
  const int8_t* G;
  const float* SG;
  const int8_t* X;
  const float* SX;
  int rows, cols, layout, wgs;
  const float* gamma;
  LayerNormBwdRows all;
};
template <bool PARTIALS>
__device__ __forceinline__ LayerNormRows first_arguments(const int8_t* X, const float* SX, const float* first, const float* second, int rows, int cols, int layout) {
  LayerNormRows a{};
  a.X = X, a.SX = SX, a.rows = rows, a.cols = cols, a.strips = layout & 255, a.teams = layout >> 8 & 255;
  if (PARTIALS) a.row_mean = first, a.row_sumsq = second;
  else a.gamma = first, a.beta = second;
  return a;
}
template <bool PARTIALS>
__device__ __forceinline__ void other_arguments(LayerNormRows& a) {
  const auto& k = kernel_arguments_from_here<LayerNormRowsArgs>()->all;
  if (PARTIALS) a.gamma = k.gamma, a.beta = k.beta;
  a.eps = k.eps, a.Y = k.Y, a.SY = k.SY, a.mean = k.mean, a.rstd = k.rstd, a.inv_cols = k.inv_cols, a.inv_blocks = k.inv_blocks;
}
__device__ __forceinline__ LayerNormBwdRows first_arguments(const int8_t* G, const float* SG, const int8_t* X, const float* SX, int rows, int cols, int layout,
                                                            int wgs, const float* gamma) {
  LayerNormBwdRows a{};
  a.G = G, a.SG = SG, a.X = X, a.SX = SX, a.rows = rows, a.cols = cols, a.strips = layout & 255, a.teams = layout >> 8 & 255, a.row_wgs = wgs, a.gamma = gamma;
  return a;
}
__device__ __forceinline__ void other_arguments(LayerNormBwdRows& a) {
  const auto& k = kernel_arguments_from_here<LayerNormBwdRowsArgs>()->all;
  a.mean = k.mean, a.rstd = k.rstd, a.dX = k.dX, a.SdX = k.SdX, a.partials = k.partials, a.dgamma = k.dgamma, a.dbeta = k.dbeta, a.inv_cols = k.inv_cols;
}

// Whether the one-pass kernels take a pass, and their launches.  The backward one returns the number of partial rows of
// dgamma | dbeta that it leaves in `partials` (at most 256 and at most rows / 32), or 0 if it has written dgamma and dbeta
// themselves, which it does not do where an output shares memory with an input (in_place).
// A block row has to fit sixteen waves.  At block sizes 64 and 128 its workgroup is long, and few of them leave compute units idle that
// the two-kernel scheme fills with tiles; backward, more than 2048 rows need another launch for the partial rows.  Two kernels -> one pass in
// us (profiles/kernel_choice.txt): forward on sixteen waves 64 block rows 7.1 -> 7.7, 128 8.6 -> 8.0, on fewer 1024 x 768 8.7 -> 6.5;
// backward 128 block rows 14.4 -> 16.0, 160 16.5 -> 14.1, up to 2048 rows twelve waves 9.9 -> 8.2, sixteen 9.3 -> 10.6.
inline bool layernorm_rows_fits(int64_t N, int64_t C, int32_t block, bool backward) {
  const int64_t waves = (C + 127) / 128 * (block / 32), block_rows = N / block;
  if (waves > 16 || block == 32) return waves <= 16;
  if (backward) return N > 2048 ? block_rows >= 160 : waves <= 12;
  return waves <= 12 || block_rows >= 128;
}
void launch_layernorm_rows_b32(const LayerNormRows& a, hipStream_t st);
void launch_layernorm_rows_b64(const LayerNormRows& a, hipStream_t st);
void launch_layernorm_rows_b128(const LayerNormRows& a, hipStream_t st);
int launch_layernorm_bwd_rows_b32(const LayerNormBwdRows& a, bool in_place, hipStream_t st);
int launch_layernorm_bwd_rows_b64(const LayerNormBwdRows& a, bool in_place, hipStream_t st);
int launch_layernorm_bwd_rows_b128(const LayerNormBwdRows& a, bool in_place, hipStream_t st);

// How many workgroups share a row group at block size 32 (jf_layernorm_split.hip), 1: the one-pass kernels.  Not where an output shares
// memory with an input, which the other workgroups of a group still read.  Every workgroup needs a compute unit to itself, backward four
// of them with those that own columns (32 each, behind the rows' workgroups, which come in eights); forward four parts pay for half the
// chip only.  One workgroup, two, four in us: forward 1024 x 1280 6.65, 5.68, 5.36; 1536 x 768 5.42, 4.72, 4.83; 4096 x 768 5.58, 4.94, 6.5;
// 6144 x 768 5.71, 6.69, 7.6; backward 1056 x 800 6.6, 6.1, 5.9; 1536 x 1536 8.6, 8.25, 8.05; 2048 x 2048 12.1, 10.05, 15; 4096 x 768 9.4, 8.4;
// 4096 x 2048 15.8, 13.75.
inline int layernorm_split_parts(int64_t N, int64_t C, bool backward) {
  const int64_t groups = backward ? (N / 32 + 7) / 8 * 8 : N / 32, units = 256 - (backward ? C / 32 : 0);
  if (C > 2048) return 1;
  return 4 * groups <= (backward ? units : 128) ? 4 : 2 * groups <= (backward ? 256 : units) ? 2 : 1;
}
// Backward: whether the two workgroups of a group leave the sums of their columns as partial rows, for another launch, instead of to workgroups
// that own columns: where there is no room for those, and where they take longer than the rows, which is by the row groups that
// each of their waves has (as many waves as strips, at least eight).  Columns apart -> partial rows in us: 2048 x 768 8.55 -> 8.95, x 1280 9.3 ->
// 11.05; 2560 x 768 10.1 -> 9.25, x 1024 8.6 -> 9.5; 2688 x 768 10.55 -> 9.45, x 1536 12.1 -> 12.15, x 2048 12.5 -> 14.0; 3072 x 768 11.9 -> 9.6, x 1536 13.6 ->
// 12.3, x 2048 13.9 -> 14.2; 3840 x 512 13.7 -> 8.45.  (One line for all widths: at 2560 rows 768 columns would gain 0.85 on its other side,
// 1024 lose 0.85.  One workgroup to a group, before: 2560 x 768 10.7, x 1024 11.1.)
inline bool layernorm_split_columns(int64_t N, int64_t C) {
  return 2 * ((N / 32 + 7) / 8 * 8) > 256 - C / 32 || (N / 32 > 80 && C <= 1536);
}
void launch_layernorm_split(LayerNormRows a, hipStream_t st);
int launch_layernorm_bwd_split(LayerNormBwdRows a, hipStream_t st);   // returns as those above

// Whether the kernels for wider rows (jf_layernorm_wide.hip) take a pass at block size 32, and their launches; the backward one
// returns its number of partial rows (at most 256 and at most rows / 32).  Forward not from the row partials of an Add: those say what
// the first of the two kernels reads the codes for.  A compute unit takes whole row groups: few of them, or a last round that is nearly
// empty, leave too many idle.  Two kernels -> one in us (profiles/kernel_choice.txt): backward 128 groups 23.2 -> 29.5, 160 24.9 -> 22.2, 256
// 43.8 -> 34.6, 320 55.4 -> 58.8, 352 44.0 -> 39.7; forward 300 groups 25.3 -> 26.8, 640 43.7 -> 41.3, 8192 x 7168 31.6 -> 27.7, x 8192 40.1 -> 42.0.
// Beyond kLayerNormWideCols LDS has room for the column sums of few waves only.
constexpr int kLayerNormWideCols = 11264;
inline bool layernorm_wide_fits(int64_t N, int64_t C, int32_t block, bool backward) {
  const int64_t groups = N / 32, room = (groups + 255) / 256 * 256;   // row groups of full rounds
  if (block != 32 || C > (backward ? kLayerNormWideCols : 7168) || groups < 160) return false;
  return room == 256 || (backward ? 3 * groups >= 2 * room : 5 * groups >= 4 * room);
}
void launch_layernorm_wide(LayerNormRows a, hipStream_t st);
int launch_layernorm_bwd_wide(LayerNormBwdRows a, hipStream_t st);

}  // namespace jf
