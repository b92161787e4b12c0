// What the LayerNorm sources share: jf_layernorm.hip (entry points; sums kernels + operators on tiles), jf_layernorm_rows.hpp (one
// pass over whole rows) and jf_layernorm_wide.hip (the same for wider rows).
#pragma once
#include "jf_rowops.hpp"

namespace jf {

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

// Whether the one-pass kernels take a pass, and their launches.  The backward one returns the number of partial rows of
// dgamma | dbeta that it leaves in `partials` (at most 256 and at most rows / 32), or 0 if it has written dgamma and dbeta
// themselves, which it does not do where an output shares memory with an input (in_place).
// A block row has to fit sixteen waves.  At block sizes 64 and 128 its workgroup is long, and few of them leave compute units
// idle that the two-kernel scheme fills with tiles.  Forward, two kernels -> one pass in us:
//   sixteen waves   8192 x 512 at block 128 (64 block rows) 7.1 -> 7.7, 8192 x 1024 at 64 (128) 8.6 -> 8.0, 24576 x 1024 17.2 -> 14.8
//   fewer           1024 x 768 at 64 8.7 -> 6.5, 4096 x 256 at 128 8.6 -> 5.4, 262144 x 768 at 64 102 -> 79, 262144 x 384 at 128 51 -> 40
// Backward, where more than 2048 rows need the launch that adds the partial rows:
//   more than 2048 rows   8192 x 384 at 128 (64) 10.3 -> 13.1, 8192 x 896 at 64 (128) 14.4 -> 16.0, 10240 x 768 (160) 16.5 -> 14.1,
//                         12288 x 1024 (192) 20.5 -> 19.3, 262144 x 768 200 -> 142, 262144 x 512 at 128 132 -> 97
//   up to 2048            1024 x 768 at 64 (twelve waves) 9.9 -> 8.2, 2048 x 256 at 128 8.9 -> 7.0; sixteen: 1024 x 512 at 128 9.3 -> 10.6
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


// Whether the kernels for wider rows (jf_layernorm_wide.hip) take a pass at block size 32, and their launches; the backward one
// returns its number of partial rows (at most 256 and at most rows / 32).  Forward not from the row partials of an Add: those say what
// the first of the two kernels reads the codes for.  A compute unit takes whole row groups: few of them, or a last round that is nearly
// empty, leave too many idle.  Two kernels -> one in us:
//   backward   4096 x 4096 (128 groups) 24.6 -> 29.5, 5120 x 2560 (160) 29.1 -> 22.2, 5120 x 4096 34.8 -> 30.6, 8192 x 4096 46.1 -> 35.3,
//              8256 x 4096 (258) 53.5 -> 55.0, 10240 x 4096 (320) 58.6 -> 56.2, 18432 x 2560 (576) 70.1 -> 56.8, 8192 x 11008 148 -> 99;
//              beyond kLayerNormWideCols LDS has room for the column sums of few waves only
//   forward    4096 x 4096 12.8 -> 13.4, 5120 x 2560 11.7 -> 9.9, 8192 x 3072 15.5 -> 12.3, 8256 x 4096 22.4 -> 25.8, 9600 x 4096 (300) 25.3 -> 26.8,
//              18432 x 2560 27.5 -> 28.6, 20480 x 4096 (640) 43.7 -> 41.3, 22528 x 3072 (704) 36.1 -> 32.3, 25600 x 2560 (800) 36.6 -> 38.9,
//              8192 x 7168 31.6 -> 27.7, 8192 x 8192 40.1 -> 42.0
constexpr int kLayerNormWideCols = 11264;
inline bool layernorm_wide_fits(int64_t N, int64_t C, int32_t block, bool backward) {
  const int64_t groups = N / 32, room = (groups + 255) / 256 * 256;   // row groups of full rounds
  if (block != 32 || C > (backward ? kLayerNormWideCols : 7168) || groups < 160) return false;
  return room == 256 || (backward ? 8 * groups >= 5 * room : 5 * groups >= 4 * room);
}
void launch_layernorm_wide(LayerNormRows a, hipStream_t st);
int launch_layernorm_bwd_wide(LayerNormBwdRows a, hipStream_t st);

}  // namespace jf
