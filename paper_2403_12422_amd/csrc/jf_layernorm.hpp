// What the two LayerNorm sources share: jf_layernorm.hip (entry points; sums kernels + operators on tiles) and
// jf_layernorm_rows.hip (one pass over whole rows).
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

// Whether the one-pass kernels take rows of C columns at this block size, and their launches.  The backward one returns
// the number of partial rows of dgamma | dbeta that it leaves in `partials` (at most 256 and at most rows / 32), or 0 if it
// has written dgamma and dbeta themselves, which it does not do where an output shares memory with an input (in_place).
bool layernorm_rows_fits(int64_t C, int32_t block);
void launch_layernorm_rows(LayerNormRows a, hipStream_t st);
int launch_layernorm_bwd_rows(LayerNormBwdRows a, bool in_place, hipStream_t st);

}  // namespace jf
