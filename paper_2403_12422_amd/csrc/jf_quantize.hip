// jf_quantize_block: per-block quantizer Q of Sec. 4, Eq. 1 (FP32/FP16 -> INT8 + FP32 scale grid).
//
// HBM-bound: 4 (or 2) bytes in, 1 byte out per element.  A workgroup of four waves owns a 128 x 128 tile; wave w owns the
// 32-row strip w of it.  Inside a strip a lane holds 16 bytes (4 FP32 or 8 FP16 columns) of 16 or 8 rows, so each row
// of the strip is read as one run of 512 or 256 bytes and written as one 128-byte line of codes.  A small tensor gives a
// compute unit a wave or two of that kind, whose 64 elements a lane are a serial chain of loads and roundings with nothing beside
// it; there the strips are narrower (launch_quantize).
#include "jf_common.hpp"

namespace jf {

__device__ __forceinline__ void load_vec(const float* p, float (&v)[4]) {
  float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void load_vec(const _Float16* p, float (&v)[8]) {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  h8 t = *reinterpret_cast<const h8*>(p);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (float)t[i];
}

// B = quantization block; a workgroup's tile is WR x WC waves of 32 rows and COLS columns each.
template <typename T, int B, bool TRANSPOSED_COPY, int WR, int WC, int COLS, StorePolicy SP>
__global__ void __launch_bounds__(64 * WR * WC) quantize_kernel(const T* __restrict__ x, int64_t ldx, int rows, int cols,
                                                        int8_t* __restrict__ q, int64_t ldq, float* __restrict__ s,
                                                        int8_t* __restrict__ qT, int64_t ldqT, float* __restrict__ sT) {
  constexpr int TR = 32 * WR, TC = COLS * WC;          // the tile
  static_assert(TR >= B || B == 32, "a block lies inside one workgroup's tile");
  static_assert(TC >= B && (!TRANSPOSED_COPY || (TR == 128 && COLS == 128 && WC == 1)), "whole blocks; the transposed copy goes by 128 x 128");
  __shared__ float s_amax[WR][TC / 32];                // [32-row strip][32-col group]
  __shared__ __align__(16) uint8_t s_codes[TRANSPOSED_COPY ? 128 * 132 : 16];
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) % WR, across = WC == 1 ? 0 : (threadIdx.x >> 6) / WR;
  const TileIndex wg = tile_of_workgroup((cols + TC - 1) / TC);
  const int r0 = (wg.y * WR + wave) * 32;              // first row of this wave's strip
  const int c0 = wg.x * TC;
  constexpr int VEC = 16 / sizeof(T), LPR = COLS / VEC, RPI = 64 / LPR, NI = 32 / RPI;   // columns per lane, lanes per row, rows at once
  const int cl = lane % LPR + LPR * across, rh = lane / LPR;
  const int col = c0 + VEC * cl, cg = cl / (32 / VEC); // first column; 32-column group of the tile
  const bool col_ok = col < cols;                      // cols % 32 == 0: the lanes of a group are in or out together

  float v[NI][VEC];
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int row = r0 + RPI * i + rh;
    if (col_ok && row < rows) {
      load_vec(x + (int64_t)row * ldx + col, v[i]);
    } else {
#pragma unroll
      for (int k = 0; k < VEC; ++k) v[i][k] = 0.0f;
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int k = 0; k < VEC; ++k) amax = fmaxf(amax, fabsf(v[i][k]));
  // lanes sharing a 32-column group: the lanes of the group in a row, and those of the rows read at once
  constexpr int GROUP_MASK = (32 / VEC - 1) | (63 & ~(LPR - 1));
  const bool group_first = (lane & GROUP_MASK) == 0;
  amax = wave_group_max<GROUP_MASK>(amax);
  if (B > 32) {  // at B = 32 a block lies inside one wave's strip: no exchange, the waves run independently
    if (group_first) s_amax[wave][cg] = amax;
    __syncthreads();
    constexpr int G = B / 32;  // 32-granules per block side
    const int w0 = (wave / G) * G, g0 = (cg / G) * G;
    amax = 0.0f;
#pragma unroll
    for (int a = 0; a < G; ++a)
#pragma unroll
      for (int b = 0; b < G; ++b) amax = fmaxf(amax, s_amax[w0 + a][g0 + b]);
  }
  float scale;
  double inv;
  block_scale(amax, scale, inv);

  const int lr = rows / B, lc = cols / B;
  // one lane per block writes the scale: the top-left 32-granule of the block
  if (group_first && col_ok && r0 < rows && (r0 % B) == 0 && ((c0 + 32 * cg) % B) == 0) {
    const int bi = r0 / B, bj = (c0 + 32 * cg) / B;
    store_scale<SP>(&s[(int64_t)bi * lc + bj], scale);
    if (TRANSPOSED_COPY) store_scale<SP>(&sT[(int64_t)bj * lr + bi], scale);
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int row = r0 + RPI * i + rh;
    uint32_t packed[VEC / 4];
#pragma unroll
    for (int k = 0; k < VEC / 4; ++k)
      packed[k] = quantize4(v[i][4 * k], v[i][4 * k + 1], v[i][4 * k + 2], v[i][4 * k + 3], inv);
    if (col_ok && row < rows) {
      if constexpr (VEC == 4) store_as<SP>(q + (int64_t)row * ldq + col, packed[0]);
      else store_as<SP>(q + (int64_t)row * ldq + col, v2i{(int)packed[0], (int)packed[1]});
    }
    if (TRANSPOSED_COPY) {
#pragma unroll
      for (int k = 0; k < VEC / 4; ++k) *reinterpret_cast<uint32_t*>(&s_codes[(wave * 32 + RPI * i + rh) * 132 + VEC * cl + 4 * k]) = packed[k];
    }
  }
  if (TRANSPOSED_COPY) {
    __syncthreads();
    // thread -> (tile column tc, 16-row chunk ch): gathers a column run and writes 16 bytes of qT
    for (int e = threadIdx.x; e < 128 * 8; e += 256) {
      const int tc = e >> 3, ch = e & 7;
      const int gc = c0 + tc, gr = wg.y * 128 + 16 * ch;
      if (gc < cols && gr < rows) {  // rows % 32 == 0: a 16-row chunk is entirely in or out
        uint32_t w[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          uint32_t acc = 0;
#pragma unroll
          for (int b = 0; b < 4; ++b) acc |= (uint32_t)s_codes[(16 * ch + 4 * d + b) * 132 + tc] << (8 * b);
          w[d] = acc;
        }
        store_part(qT + (int64_t)gc * ldqT + gr, make_uint4(w[0], w[1], w[2], w[3]));
      }
    }
  }
}

// Narrow strips, in workgroups of one block row and, at block size 128, one block: 64 columns a wave up to 256 tiles of 128 x 128, one
// for each compute unit (FP16, half the bytes in flight a lane, up to 768); 32 columns for the smallest tensors and, in FP16 at block
// sizes 64 and 128, up to 256 tiles.  Beyond, the waves fill the chip as they are and narrower ones only take more instructions.  With 128,
// 64 and 32 columns in us: FP32 at block 32 63 tiles 4.1, 3.4, 3.2, 192 tiles 5.6, 5.0, 5.8, 384 tiles 6.3, 6.8, 7.7; FP16 768 tiles 10.7, 10.1,
// 15.0, 1024 tiles 13.3, 14.0 (profiles/kernel_choice.txt).
template <typename T, int B>
static void launch_quantize(const T* x, int64_t ldx, int rows, int cols, int8_t* q, int64_t ldq, float* s, int8_t* qT,
                            int64_t ldqT, float* sT, hipStream_t st) {
  // the kernel for tiles of WR x WC strips of COLS columns
  const auto launch = [&](auto kernel, int WR, int WC, int COLS) {
    const dim3 grid(tile_grid((cols + COLS * WC - 1) / (COLS * WC), (rows + 32 * WR - 1) / (32 * WR)));
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WR * WC), 0, st, x, ldx, rows, cols, q, ldq, s, qT, ldqT, sT);
  };
  constexpr bool FP16 = sizeof(T) == 2;
  const int64_t tiles = (int64_t)((cols + 127) / 128) * ((rows + 127) / 128);
  with_store_policy(rows, ldq, [&](auto sp) {
    constexpr StorePolicy SP = decltype(sp)::value;
    if (qT) return launch(quantize_kernel<T, B, true, 4, 1, 128, SP>, 4, 1, 128);
    if constexpr (SP == kStoreThrough) {
      constexpr int G = B / 32;
      if constexpr (B == 32 || FP16)
        if (tiles <= (B == 32 ? 64 : 256)) return launch(quantize_kernel<T, B, false, G, G, 32, SP>, G, G, 32);
      if (tiles <= (FP16 ? 768 : 256)) return launch(quantize_kernel<T, B, false, G, (B + 63) / 64, 64, SP>, G, (B + 63) / 64, 64);
    }
    launch(quantize_kernel<T, B, false, 4, 1, 128, SP>, 4, 1, 128);
  });
}

template <typename T>
static void dispatch_quantize(int block, const T* x, int64_t ldx, int rows, int cols, int8_t* q, int64_t ldq, float* s,
                              int8_t* qT, int64_t ldqT, float* sT, hipStream_t st) {
  if (block == 32) launch_quantize<T, 32>(x, ldx, rows, cols, q, ldq, s, qT, ldqT, sT, st);
  else if (block == 64) launch_quantize<T, 64>(x, ldx, rows, cols, q, ldq, s, qT, ldqT, sT, st);
  else launch_quantize<T, 128>(x, ldx, rows, cols, q, ldq, s, qT, ldqT, sT, st);
}

// Dequantizer Q^-1 of Eq. 1: out = code * scale as FP32 or FP16 (the hand-over to a floating-point operator
// such as the FP16 attention core of Sec. 7.1).  HBM-bound: 1 byte in, 2 or 4 out per element.  A thread writes 16 bytes
// (8 FP16 or 4 FP32 values) at a time, so that a wave fills whole lines, and takes DQ_CHUNKS such chunks 256 apart, whose
// codes and scales are requested before the first is used; rows follow each other without a gap, so that no lane idles at
// their ends.  The quotient chunk / (chunks per row) is formed once per workgroup in 64 bits and per chunk in 32.
static constexpr int DQ_CHUNKS = 4;
template <typename T, StorePolicy SP>
__global__ void __launch_bounds__(256) dequantize_kernel(const int8_t* __restrict__ q, const float* __restrict__ s, int rows,
                                                          int cols, int block_log2, T* __restrict__ out, int64_t ldo) {
  constexpr int VEC = 16 / sizeof(T);
  typedef typename std::conditional<VEC == 8, uint2, uint32_t>::type packed_t;
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  const uint32_t chunks = cols / VEC;
  const int64_t first = (int64_t)blockIdx.x * (256 * DQ_CHUNKS), total = (int64_t)rows * chunks;
  const int row0 = (int)(first / chunks);
  const uint32_t rem = (uint32_t)(first - (int64_t)row0 * chunks);
  const int lc = cols >> block_log2;
  packed_t p[DQ_CHUNKS];
  float sc[DQ_CHUNKS];
  int row[DQ_CHUNKS], col[DQ_CHUNKS];
#pragma unroll
  for (int u = 0; u < DQ_CHUNKS; ++u) {
    const uint32_t i = rem + u * 256 + threadIdx.x, r = i / chunks;
    row[u] = row0 + (int)r;
    col[u] = VEC * (int)(i - r * chunks);
    if (first + u * 256 + threadIdx.x < total) {
      p[u] = *reinterpret_cast<const packed_t*>(q + (int64_t)row[u] * cols + col[u]);
      sc[u] = s[(int64_t)(row[u] >> block_log2) * lc + (col[u] >> block_log2)];
    }
  }
#pragma unroll
  for (int u = 0; u < DQ_CHUNKS; ++u) {
    if (first + u * 256 + threadIdx.x >= total) break;
    vec_t v;
#pragma unroll
    for (int b = 0; b < VEC; ++b) {
      uint32_t w;
      if constexpr (VEC == 8) w = b < 4 ? p[u].x : p[u].y;
      else w = p[u];
      v[b] = (T)(byte_to_float(w, b & 3) * sc[u]);
    }
    store_as<SP>(out + (int64_t)row[u] * ldo + col[u], v);
  }
}

}  // namespace jf

extern "C" int32_t jf_dequantize_block(const int8_t* q, const float* s, int64_t rows, int64_t cols, int32_t block,
                                       void* out, int32_t out_dtype, int64_t ldo, void* stream) {
  using namespace jf;
  if (!q || !s || !out) return JF_ERR_NULL;
  if (out_dtype != 0 && out_dtype != 1) return JF_ERR_DTYPE;
  if (!valid_block(block)) return JF_ERR_BLOCK;
  if (!valid_dim(rows, block) || !valid_dim(cols, block) || !valid_size(rows, cols) || ldo < cols) return JF_ERR_SHAPE;
  if (!aligned16(q) || !aligned4(s) || !aligned16(out) || (ldo % 8)) return JF_ERR_ALIGN;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int64_t per_wg = 256 * DQ_CHUNKS * (out_dtype == 0 ? 4 : 8);
  const unsigned grid = (unsigned)((rows * cols + per_wg - 1) / per_wg);
  with_store_policy(rows, ldo * (out_dtype == 0 ? 4 : 2), [&](auto sp) {
    constexpr StorePolicy SP = decltype(sp)::value;
    if (out_dtype == 0)
      hipLaunchKernelGGL((dequantize_kernel<float, SP>), dim3(grid), dim3(256), 0, st, q, s, (int)rows, (int)cols, block_log2(block),
                         static_cast<float*>(out), ldo);
    else
      hipLaunchKernelGGL((dequantize_kernel<_Float16, SP>), dim3(grid), dim3(256), 0, st, q, s, (int)rows, (int)cols, block_log2(block),
                         static_cast<_Float16*>(out), ldo);
  });
  return launch_status();
}

extern "C" int32_t jf_quantize_block(const void* x, int32_t x_dtype, int64_t rows, int64_t cols, int64_t ldx,
                                     int32_t block, int8_t* q, int64_t ldq, float* s, int8_t* qT, int64_t ldqT,
                                     float* sT, void* stream) {
  using namespace jf;
  if (!x || !q || !s) return JF_ERR_NULL;
  if ((qT == nullptr) != (sT == nullptr)) return JF_ERR_NULL;
  if (x_dtype != 0 && x_dtype != 1) return JF_ERR_DTYPE;
  if (!valid_block(block)) return JF_ERR_BLOCK;
  if (!valid_dim(rows, block) || !valid_dim(cols, block) || !valid_size(rows, cols)) return JF_ERR_SHAPE;
  if (ldx < cols || ldq < cols || (qT && ldqT < rows)) return JF_ERR_SHAPE;
  if (!aligned16(x) || !aligned16(q) || !aligned4(s) || (ldx % 16) || (ldq % 16)) return JF_ERR_ALIGN;
  if (qT && (!aligned16(qT) || !aligned4(sT) || (ldqT % 16))) return JF_ERR_ALIGN;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (x_dtype == 0)
    dispatch_quantize<float>(block, static_cast<const float*>(x), ldx, (int)rows, (int)cols, q, ldq, s, qT, ldqT, sT, st);
  else
    dispatch_quantize<_Float16>(block, static_cast<const _Float16*>(x), ldx, (int)rows, (int)cols, q, ldq, s, qT, ldqT, sT, st);
  return launch_status();
}
