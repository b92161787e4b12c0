// Helpers shared by the INT8-in / INT8-out operators (Sec. 6, Alg. 2, App. A): unpacking and Eq. 1 for 16 codes at a
// time, the lane mapping of the strip kernels, and host-side argument checks.
#pragma once
#include "jf_common.hpp"

namespace jf {

__device__ __forceinline__ uint4 quantize16(const float (&y)[16], double inv) {
  uint4 o;
  o.x = quantize4(y[0], y[1], y[2], y[3], inv);
  o.y = quantize4(y[4], y[5], y[6], y[7], inv);
  o.z = quantize4(y[8], y[9], y[10], y[11], inv);
  o.w = quantize4(y[12], y[13], y[14], y[15], inv);
  return o;
}

// 16 codes -> (code + 128) as float: one XOR per dword flips the sign bits, then each byte converts
// with v_cvt_f32_ubyteN.  The caller folds the -128 into its fused multiply-add.
__device__ __forceinline__ void unpack16_biased(const uint4& p, float (&u)[16]) {
  const uint32_t w[4] = {p.x ^ 0x80808080u, p.y ^ 0x80808080u, p.z ^ 0x80808080u, p.w ^ 0x80808080u};
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    u[4 * d + 0] = (float)(w[d] & 0xffu);
    u[4 * d + 1] = (float)((w[d] >> 8) & 0xffu);
    u[4 * d + 2] = (float)((w[d] >> 16) & 0xffu);
    u[4 * d + 3] = (float)(w[d] >> 24);
  }
}

// ------------------------------------------------------------------------------------------------
// The element-wise operators on strips.  A wave owns a strip of 32 rows x 128 columns.  Lane l = (rsub = l / 8, ch = l % 8)
// holds the 16-byte chunk ch of rows rsub, rsub + 8, rsub + 16, rsub + 24 of the strip: every load or store instruction of
// the wave moves eight full 128-byte lines, and a lane's 64 elements belong to ONE quantization block.  At block size 32 the
// strip is four blocks side by side: their max-abs is a local maximum followed by four cross-lane steps, and nothing is
// exchanged between waves, no barrier.  At block sizes 64 and 128 two or four waves of a workgroup stand one above the other
// and exchange it through LDS.  Per element the kernels spend what Alg. 2 needs (unpack, the operator, max-abs, Eq. 1) and
// little else; the per-lane overhead is paid once per 64 elements.
// RW = 16: waves of 16 rows, twice as many one above the other (block size 32 exchanges its max-abs like the others then): half the
// serial chain of a wave, and still whole lines.  (Strips of 64 columns and 32 rows do as well while everything is in a cache, but their
// 64-byte pieces cost a third of the memory's bandwidth: GELU 8192 x 2048 8.0 -> 11.1 us from memory, 8.4 -> 7.7 from the cache.)
// Waves per workgroup: at block size 32 four neighbouring strips of the same rows, so that 512 contiguous bytes of every row
// are requested close together in time (on 0.8 GB tensors of 3072 columns 5.4-5.7 TB/s instead of 4.4-5.0 with one strip per
// workgroup); two by two at 64 and one above the other at 128, and twice as wide for results that go to memory (262144 x
// 3072, four and eight waves: Add at 64 449 and 424 us, at 128 495 and 447, Dropout 323 and 301, 368 and 318; 8192 x 1280 Add
// 6.7 and 7.2, GELU backward at 128 7.7 and 8.7).
constexpr int kStripWaves = 4;
constexpr int strip_waves(int block, StorePolicy sp) { return block == 32 || sp == kStoreThrough ? 4 : 8; }
template <int B, int WAVES = kStripWaves, int RW = 32>
struct Strip {
  static constexpr int BT = B / RW;        // waves that share a block
  static constexpr int PASSES = RW / 8;    // passes of eight rows
  int ch, rsub;     // chunk column and row of the lane inside an 8-row pass
  int bi, lc;       // RW-row group of the strip, block columns of the matrix
  int c0, col;      // first column of the strip, first column of the lane's chunks
  bool ok;          // the lane's chunks lie inside the matrix (cols % 32 == 0: a block is all in or all out)
  int64_t base;     // element offset of the lane's chunk in pass 0; pass p adds 8 p cols.  Lanes outside the matrix
                    // point at the strip's first chunk instead: they load like the others (no branch), share their
                    // reductions only with each other (whole blocks are in or out), and store nothing.
  int lane, wave;   // lane of the wave, wave of the workgroup
  bool inside;      // the wave's strip exists (the last workgroup may hold fewer; the others repeat the last strip)
  __device__ __forceinline__ Strip(int rows, int cols, unsigned first = 0) {   // first: workgroups before the strips
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ch = lane & 7;
    rsub = lane >> 3;
    const unsigned groups = (unsigned)((cols + 127) / 128), strips = groups * (unsigned)(rows / B);
    const unsigned id = (blockIdx.x - first) * (WAVES / BT) + wave / BT;   // numbered column group fastest
    inside = id < strips;
    const unsigned sid = inside ? id : strips - 1;
    c0 = (int)(sid % groups) * 128;
    bi = (int)(sid / groups) * BT + wave % BT;
    lc = cols / B;
    col = c0 + 16 * ch;
    ok = col < cols;
    base = (int64_t)(bi * RW + rsub) * cols + (ok ? col : c0);
    if (BT > 1) ok = ok && inside;   // with BT == 1 a wave that is not inside ends at once
  }
  // index of the lane's block in a scale grid (clamped like base), and whether the lane is the one to store its scale
  __device__ __forceinline__ int64_t block_index() const { return (int64_t)(bi / BT) * lc + (col < lc * B ? col : c0) / B; }
  __device__ __forceinline__ bool owns_scale() const { return (lane & (56 | (B / 16 - 1))) == 0 && (BT == 1 || wave % BT == 0); }
};

typedef Strip<32> Strip32;

// Block max-abs, over the lanes of a strip that share a block column and over the waves that share the block through `exchange`
// (up to four values per wave).  At block sizes 64 and 128 every wave of the workgroup has to get here.
template <int B, int WAVES, int RW>
__device__ __forceinline__ float strip_block_max(float m, const Strip<B, WAVES, RW>& t, float (*exchange)[4]) {
  m = wave_group_max<56 | (B / 16 - 1)>(m);
  if constexpr (B > RW) {
    if ((t.lane & (56 | (B / 16 - 1))) == 0) exchange[t.wave][t.ch / (B / 16)] = m;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < t.BT; ++k) m = fmaxf(m, exchange[t.wave / t.BT * t.BT + k][t.ch / (B / 16)]);
  }
  return m;
}
// the same and Eq. 1's scale
template <int B, int WAVES, int RW>
__device__ __forceinline__ void strip_block_scale(float m, const Strip<B, WAVES, RW>& t, float (*exchange)[4], float& scale, double& inv) {
  block_scale(strip_block_max(m, t, exchange), scale, inv);
}
// at block size 32: the 16 lanes of a strip that share a block column (same ch / 2)
__device__ __forceinline__ void strip32_block_scale(float m, float& scale, double& inv) { block_scale(wave_group_max<56 | 1>(m), scale, inv); }

__device__ __forceinline__ void load16f(const float* p, float (&v)[16]) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const float4 t = *reinterpret_cast<const float4*>(p + 4 * d);
    v[4 * d] = t.x; v[4 * d + 1] = t.y; v[4 * d + 2] = t.z; v[4 * d + 3] = t.w;
  }
}

// ------------------------------------------------------------------------------------------------ host
// workgroups of the strip kernels: WAVES strips of 32 rows each
template <int B = 32, int WAVES = kStripWaves, int RW = 32>
static inline dim3 strip_grid(int64_t rows, int64_t cols) {
  const int64_t strips = ((cols + 127) / 128) * (rows / B), per_wg = WAVES * RW / B;
  return dim3((unsigned)((strips + per_wg - 1) / per_wg));
}
// f(integral_constant<int, B>) for a block size
template <class F>
static inline void with_block(int block, F&& f) {
  if (block == 32) f(std::integral_constant<int, 32>());
  else if (block == 64) f(std::integral_constant<int, 64>());
  else f(std::integral_constant<int, 128>());
}

// f(block size, waves per workgroup, rows of a wave, store policy) as integral constants: 16 rows instead of 32 if `low`, for results
// that are written through; at block size 128 only for an operator that has such waves there (LOW128)
template <bool LOW128, class F>
static void with_instance(int block, int64_t rows, int64_t cols, bool low, F&& f) {
  with_block(block, [&](auto b) {
    with_store_policy(rows, cols, [&](auto sp) {
      constexpr int B = decltype(b)::value;
      constexpr StorePolicy SP = decltype(sp)::value;
      if constexpr (SP == kStoreThrough && (B < 128 || LOW128))
        if (low) return f(b, std::integral_constant<int, B == 128 ? 8 : 4>(), std::integral_constant<int, 16>(), sp);
      f(b, std::integral_constant<int, strip_waves(B, SP)>(), std::integral_constant<int, 32>(), sp);
    });
  });
}

static inline int32_t check_eltwise(const void* x, const void* sx, const void* y, const void* sy, int64_t N, int64_t C,
                             int32_t block) {
  if (!x || !sx || !y || !sy) return JF_ERR_NULL;
  if (!valid_block(block)) return JF_ERR_BLOCK;
  if (!valid_dim(N, block) || !valid_dim(C, block) || !valid_size(N, C)) return JF_ERR_SHAPE;
  if (!aligned16(x) || !aligned4(sx) || !aligned16(y) || !aligned4(sy)) return JF_ERR_ALIGN;
  return JF_OK;
}

}  // namespace jf
