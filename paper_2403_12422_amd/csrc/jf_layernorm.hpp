// What the two LayerNorm sources share: jf_layernorm.hip (entry points; sums kernels + operators on tiles) and
// jf_layernorm_rows.hpp (one pass over whole rows).
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

}  // namespace jf
