// jf_quantize_block: per-block quantizer Q of Sec. 4, Eq. 1 (FP32/FP16 -> INT8 + FP32 scale grid).
//
// HBM-bound: 4 (or 2) bytes in, 1 byte out per element.  A wave owns a strip of 32 rows x 128 columns, a workgroup the one, two or four strips
// of a block row one above the other.  Inside a strip a lane holds 16 bytes (4 FP32 or 8 FP16 columns) of 16 or 8 rows, so each row
// of the strip is read as one run of 512 or 256 bytes and written as one 128-byte line of codes.  A small tensor gives a
// compute unit a wave or two of that kind, whose 64 elements a lane are a serial chain of loads and roundings with nothing beside
// it; there the strips are narrower (launch_quantize).
#include "jf_common.hpp"

namespace jf {

// A lane's 16 bytes of a row, what the block's max-abs takes from the lane, and Eq. 1 for them (packed: one dword for four codes).
template <typename T>
struct Row16;

template <>
struct Row16<float> {
  static constexpr int VEC = 4;
  float4 t;
  template <int NI>
  static __device__ __forceinline__ float amax(const Row16 (&v)[NI]) {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {   // (the compiler's fmaxf quiets operands with an instruction each)
      asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v[i].t.x), "v"(v[i].t.y));
      asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v[i].t.z), "v"(v[i].t.w));
    }
    return m;
  }
  struct Scale {
    float scale;
    double inv;
    explicit __device__ __forceinline__ Scale(float amax) { block_scale(amax, scale, inv); }
  };
  __device__ __forceinline__ void codes(const Scale& s, uint32_t (&packed)[1]) const { packed[0] = quantize4(t.x, t.y, t.z, t.w, s.inv); }
};

// FP16: one FP32 FMA per element rounds the exact quotient x / s, which takes the three instructions of code_bits() for any FP32 number.
// x has 11 bits, and s is within 2^-24 of amax / 127, where amax is one of the x.  So
//   * 127 x / amax is a tie k + 1/2 or at least 1 / (254 * 2047) > 2^-19 of itself away from one (254 X and (2 k + 1) A 2^j are integers, X
//     and A the 11-bit significands), and a reciprocal that is off by 2^-22 does not take x / s past a tie that 127 x / amax is not on;
//   * where it is a tie, x / s lies beyond it if s < amax / 127 and short of it if s > amax / 127.  One ulp added to fl32(1 / s) or taken off it
//     brings the reciprocal to the side of 127 / amax that 1 / s is on, whatever its own rounding did, and with it the product;
//   * where s = amax / 127 exactly, a tie of x / s is one, and the FMA sends it to even if fl32(1 / s) = 1 / s, a power of two.  The other
//     scales (amax a multiple of 127 other than by a power of two, 7 of 1024 significands) take code_bits().
// (5.25 -> 2.75 vector instructions an element.  8192 x 1280 from memory 9.4 -> 8.2 us, 8192 x 3840 22.4 -> 18.9 = 5.0 TB/s, 32768 x 4096
// 77.1 -> 73.8 = 5.5 TB/s: the waves of a tensor this size start together, and their arithmetic follows their loads.  Hand-over of 8192 x 1280 to
// attention and back, four launches, 58.5 -> 53.6.)
template <>
struct Row16<_Float16> {
  static constexpr int VEC = 8;
  uint4 t;
  template <int NI>
  static __device__ __forceinline__ float amax(const Row16 (&v)[NI]) {
    uint32_t m = 0;
    const auto larger = [](uint32_t a, uint32_t b) __attribute__((always_inline)) {   // of two pairs (the compiler's fmax quiets its operands first)
      uint32_t r;
      asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
      return r;
    };
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t w[4] = {v[i].t.x, v[i].t.y, v[i].t.z, v[i].t.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) m = larger(m, w[k] & 0x7fff7fffu);
    }
    m = larger(m, m >> 16);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)m);
  }
  struct Scale {
    float scale, inv32;
    double inv;
    bool one_fma;   // for all blocks of the wave
    explicit __device__ __forceinline__ Scale(float amax) {
      block_scale(amax, scale, inv);
      const float over = __builtin_fmaf(scale, 127.0f, -amax);   // exact in sign: of scale - amax / 127
      const uint32_t near = __builtin_bit_cast(uint32_t, (float)inv);
      inv32 = __builtin_bit_cast(float, over > 0.0f ? near - 1 : over < 0.0f ? near + 1 : near);
      one_fma = !__any(over == 0.0f && (__builtin_bit_cast(uint32_t, scale) & 0x7fffffu));
    }
  };
  // element H of the pair in w, as code_bits() leaves it: 1.5 * 2^23 added by the FMA rounds to an integer, to even, in the low mantissa bits
  template <int H>
  static __device__ __forceinline__ uint32_t element(uint32_t w, float inv32) {
    uint32_t r;
    if constexpr (H == 0) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(inv32), "v"(12582912.0f));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(inv32), "v"(12582912.0f));
    return r;
  }
  __device__ __forceinline__ void codes(const Scale& s, uint32_t (&packed)[2]) const {
    const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t a = w[2 * k], b = w[2 * k + 1];
      if (__builtin_expect(s.one_fma, 1)) {
        packed[k] = pack_codes(element<0>(a, s.inv32), element<1>(a, s.inv32), element<0>(b, s.inv32), element<1>(b, s.inv32));
      } else {
        const auto h = [](uint32_t pair, int i) __attribute__((always_inline)) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(pair >> (16 * i))); };
        packed[k] = quantize4(h(a, 0), h(a, 1), h(b, 0), h(b, 1), s.inv);
      }
    }
  }
};

static constexpr int kTransposeBytes = 128 * 132;   // LDS of a transposed copy's tile

// B = quantization block; a workgroup's tile is WR x WC waves of 32 rows and COLS columns each.
template <typename T, int B, bool TRANSPOSED_COPY, int WR, int WC, int COLS, StorePolicy SP>
__global__ void __launch_bounds__(64 * WR * WC) quantize_kernel(const T* __restrict__ x, int64_t ldx, int rows, int cols,
                                                        int8_t* __restrict__ q, int64_t ldq, float* __restrict__ s,
                                                        int8_t* __restrict__ qT, int64_t ldqT, float* __restrict__ sT) {
  constexpr int TR = 32 * WR, TC = COLS * WC;          // the tile
  static_assert(TR >= B || B == 32, "a block lies inside one workgroup's tile");
  static_assert(TC >= B && (!TRANSPOSED_COPY || (TR == 128 && COLS == 128 && WC == 1)), "whole blocks; the transposed copy goes by 128 x 128");
  __shared__ float s_amax[WR][TC / 32];                // [32-row strip][32-col group]
  __shared__ __align__(16) uint8_t s_codes[TRANSPOSED_COPY ? kTransposeBytes : 16];
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) % WR, across = WC == 1 ? 0 : (threadIdx.x >> 6) / WR;
  const TileIndex wg = tile_of_workgroup((cols + TC - 1) / TC);
  const int r0 = __builtin_amdgcn_readfirstlane((wg.y * WR + wave) * 32);   // first row of this wave's strip
  const int c0 = wg.x * TC;
  constexpr int VEC = Row16<T>::VEC, LPR = COLS / VEC, RPI = 64 / LPR, NI = 32 / RPI;   // columns per lane, lanes per row, rows at once
  const int cl = lane % LPR + LPR * across, rh = lane / LPR;
  const int col = c0 + VEC * cl, cg = cl / (32 / VEC); // first column; 32-column group of the tile
  // rows and cols are multiples of 32: a strip and the lanes of a group are in or out together.  What is outside loads like the rest, from the
  // last strip and the tile's first columns, without a branch, and stores nothing.  (With a branch and the address of its own around each
  // load the kernel had 212 instructions for 145 at 32 columns of FP32, most of them before the loads: 0.1-0.2 us a launch.)
  const bool inside = col < cols && (WR * 32 == B || r0 < rows);

  Row16<T> v[NI];
  const T* from = x + (int64_t)(WR * 32 == B ? r0 : min(r0, rows - 32)) * ldx + ((uint32_t)rh * (uint64_t)ldx + (col < cols ? col : c0));
#pragma unroll
  for (int i = 0; i < NI; ++i, from += RPI * ldx) v[i] = *reinterpret_cast<const Row16<T>*>(from);
  float amax = Row16<T>::amax(v);
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
  const typename Row16<T>::Scale scale(amax);

  const int lr = rows / B, lc = cols / B;
  // one lane per block writes the scale: the top-left 32-granule of the block
  if (group_first && inside && (r0 % B) == 0 && ((c0 + 32 * cg) % B) == 0) {
    const int bi = r0 / B, bj = (c0 + 32 * cg) / B;
    store_scale<SP>(&s[(int64_t)bi * lc + bj], scale.scale);
    if (TRANSPOSED_COPY) store_scale<SP>(&sT[(int64_t)bj * lr + bi], scale.scale);
  }
  int8_t* to = q + (int64_t)r0 * ldq + ((uint32_t)rh * (uint64_t)ldq + col);
#pragma unroll
  for (int i = 0; i < NI; ++i, to += RPI * ldq) {
    uint32_t packed[VEC / 4];
    v[i].codes(scale, packed);
    if (inside) {
      if constexpr (VEC == 4) store_as<SP>(to, packed[0]);
      else store_as<SP>(to, v2i{(int)packed[0], (int)packed[1]});
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

// Workgroups of one block row: of one strip of 128 columns, and up to 256 tiles of 128 x 128, one for each compute unit, of strips of 64 columns
// (at block size 128 two, one block): half the serial chain of a wave, and more waves than the chip has SIMDs from 64 tiles on.  Beyond, the waves
// fill it as they are, and half lines of codes cost more.  With 128 and 64 columns from memory, us: FP16 at block 32 48 tiles 3.5, 3.0, 128 tiles
// 4.0, 3.3, 256 tiles 4.7, 4.7, 384 tiles 6.0, 6.2, 1920 tiles 19.7, 21.0; FP32 48 tiles 3.7, 2.9, 256 tiles 6.2, 6.1, 768 tiles 13.9, 14.0; block
// 64 and 128 alike.  (Strips of 32 columns are slower at all sizes: FP32 at block 32 4 tiles 2.55 for 2.35, 48 tiles 3.25 for 2.95, from the cache 2.95
// for 2.45.  Four block rows to a workgroup: FP16 8192 x 3840 20.4 for
// 19.7, FP32 4096 x 3072 14.1 for 13.9.)
//
// Results that are streamed, 64 MB and more: eight waves on a compute unit (six of FP32, which have twice the bytes in flight), where their registers
// would allow 20 to 32.  16 to 24 MB in flight are enough for the memory, and what is in flight beyond lies further apart in it.  FP16 takes two strips
// across, so that a workgroup reads 512 bytes of a row, unless the strips are few and the last workgroup's second one is none.  As many as fit -> these, us:
// FP16 1048576 x 768 440 -> 400, 262144 x 3072 443 -> 412, 32768 x 4096 74.5 -> 67, at block 128 1048576 x 768 447 -> 414; FP32 262144 x 3072 708 -> 660,
// 1048576 x 768 722 -> 690, 32768 x 4096 120 -> 115, at block 64 262144 x 3072 713 -> 682; with the transposed copy FP32 262144 x 3072 896 -> 846, FP16 621 ->
// 612, at block 64 and 128 622 -> 596.  (FP16 1048576 x 768 by one strip 416; 1048576 x 128 by two 83, by one 68.)
// FP32 with the transposed copy, from 22 M elements on: twelve waves, sixteen where rows share lines.  Without a bound the loads without branches had cost
// it 1 to 3 % from memory: 12288 x 4096 65.2 with them, 67.0, now 62.2 us; 4096 x 5632 29.4, 30.4, 29.2, from the last-level cache 22.8 each; 32768 x 1024 42.7, 43.5,
// 41.4, from the cache 31.6 each; 16384 x 2080 50.5, 51.1, 50.2; smaller ones lose 1 to 3 % from the cache by it (20480 x 1024 20.6 -> 21.25).
template <typename T, int B>
static void launch_quantize(const T* x, int64_t ldx, int rows, int cols, int8_t* q, int64_t ldq, float* s, int8_t* qT,
                            int64_t ldqT, float* sT, hipStream_t st) {
  // the kernel for tiles of WR x WC strips of COLS columns; `waves`: at most so many on a compute unit, kept to by the LDS that a workgroup asks for
  const auto launch = [&](auto kernel, int WR, int WC, int COLS, int waves = 0) {
    const dim3 grid(tile_grid((cols + COLS * WC - 1) / (COLS * WC), (rows + 32 * WR - 1) / (32 * WR)));
    const unsigned own = 2048 + (qT ? kTransposeBytes : 0);   // the kernel's own, with a margin
    const unsigned lds = waves ? kLdsBytes / (waves / (WR * WC)) - own : 0;
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WR * WC), lds, st, x, ldx, rows, cols, q, ldq, s, qT, ldqT, sT);
  };
  constexpr int G = B / 32;
  const int64_t tiles = (int64_t)((cols + 127) / 128) * ((rows + 127) / 128);
  with_store_policy(rows, ldq, [&](auto sp) {
    constexpr StorePolicy SP = decltype(sp)::value;
    if (qT) {
      const int waves = SP == kStoreStream ? 8 : sizeof(T) == 2 || int64_t(rows) * cols < 21 << 20 ? 0 : SP == kStoreThrough ? 12 : 16;
      return launch(quantize_kernel<T, B, true, 4, 1, 128, SP>, 4, 1, 128, waves);
    }
    if constexpr (SP == kStoreThrough) {
      if (tiles <= 256) return launch(quantize_kernel<T, B, false, G, (B + 63) / 64, 64, SP>, G, (B + 63) / 64, 64);
    }
    if constexpr (SP == kStoreStream) {
      const int strips = (cols + 127) / 128;
      if constexpr (sizeof(T) == 2 && B <= 64)
        if (strips % 2 == 0 || strips > 8) return launch(quantize_kernel<T, B, false, G, 2, 128, SP>, G, 2, 128, 8);
      return launch(quantize_kernel<T, B, false, G, 1, 128, SP>, G, 1, 128, sizeof(T) == 4 && B <= 64 ? 6 : 8);
    }
    launch(quantize_kernel<T, B, false, G, 1, 128, SP>, G, 1, 128);
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
// (8 FP16 or 4 FP32 values) at a time, so that a wave fills whole lines, and takes CHUNKS such chunks 256 apart, whose
// codes and scales are requested before the first is used; rows follow each other without a gap, so that no lane idles at
// their ends.  The quotient chunk / (chunks per row) is formed once per workgroup in 64 bits and per chunk in 32.
// CHUNKS: two.  More of them have more requests in flight a lane, but their addresses, 36 instructions each, stand in front of them one after the other,
// and waves of fewer come and go more evenly.  FP16 with one, two, three and four chunks, us: 8192 x 3840 18.9, 17.6, 18.0, 18.6, from the last-level
// cache 13.2, 12.6, 12.9, 12.4; 8192 x 1280 8.0, 7.8, 8.3, 8.0; 8192 x 2048 11.1, 11.2, 11.4, 12.0; 1024 x 1024 2.4, 2.3, 2.4, 2.65; 65536 x 4096
// 137, 128, 129, 130; FP32 with two and four 8192 x 1280 11.2 and 12.1, 65536 x 4096 205.5 and 206.5.  Four for FP32 from 335 M elements on, where
// it is the other way round: 131072 x 3072 311 and 308, 262144 x 3072 631 and 614, 524288 x 3072 1275 and 1239 (FP16 384 and 393, 773 and 800); and
// where two would make a grid of 2^32 threads, which cannot be launched.
template <typename T, StorePolicy SP, int CHUNKS>
__global__ void __launch_bounds__(256) dequantize_kernel(const int8_t* __restrict__ q, const float* __restrict__ s, int rows,
                                                          int cols, int block_log2, T* __restrict__ out, int64_t ldo) {
  constexpr int VEC = 16 / sizeof(T);
  typedef typename std::conditional<VEC == 8, uint2, uint32_t>::type packed_t;
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  const uint32_t chunks = cols / VEC;
  const int64_t first = (int64_t)blockIdx.x * (256 * CHUNKS), total = (int64_t)rows * chunks;
  const int row0 = (int)(first / chunks);
  const uint32_t rem = (uint32_t)(first - (int64_t)row0 * chunks);
  const int lc = cols >> block_log2;
  packed_t p[CHUNKS];
  float sc[CHUNKS];
  int row[CHUNKS], col[CHUNKS];
#pragma unroll
  for (int u = 0; u < CHUNKS; ++u) {
    const uint32_t i = rem + u * 256 + threadIdx.x, r = i / chunks;
    row[u] = row0 + (int)r;
    col[u] = VEC * (int)(i - r * chunks);
    if (first + u * 256 + threadIdx.x < total) {
      p[u] = *reinterpret_cast<const packed_t*>(q + (int64_t)row[u] * cols + col[u]);
      sc[u] = s[(int64_t)(row[u] >> block_log2) * lc + (col[u] >> block_log2)];
    }
  }
#pragma unroll
  for (int u = 0; u < CHUNKS; ++u) {
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
  with_store_policy(rows, ldo * (out_dtype == 0 ? 4 : 2), [&](auto sp) {
    constexpr StorePolicy SP = decltype(sp)::value;
    const auto launch = [&](auto kernel, auto* to, int chunks) {
      const int64_t per_wg = 256 * chunks * (int64_t)(16 / sizeof(*to));
      hipLaunchKernelGGL(kernel, dim3((unsigned)((rows * cols + per_wg - 1) / per_wg)), dim3(256), 0, st, q, s, (int)rows, (int)cols, block_log2(block), to, ldo);
    };
    const auto launch_as = [&](auto* to) {
      typedef std::remove_pointer_t<decltype(to)> T;
      constexpr int64_t VEC = 16 / sizeof(T);
      if constexpr (SP != kStoreThrough)
        if (rows * cols >= (sizeof(T) == 4 ? int64_t(320) << 20 : (int64_t(1) << 32) * 2 * VEC - 4096)) return launch(dequantize_kernel<T, SP, 4>, to, 4);
      launch(dequantize_kernel<T, SP, 2>, to, 2);
    };
    if (out_dtype == 0) launch_as(static_cast<float*>(out));
    else launch_as(static_cast<_Float16*>(out));
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
