// Shared device / host helpers of the gfx950 per-block INT8 library.
// Wavefront = 64 lanes everywhere in this file.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstddef>
#include <tuple>
#include <type_traits>

#include "jetfire.h"

namespace jf {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- host side
extern thread_local int32_t g_last_hip_error;

inline int32_t launch_status() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    g_last_hip_error = (int32_t)e;
    return JF_ERR_LAUNCH;
  }
  return JF_OK;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }
inline bool valid_block(int32_t b) { return b == 32 || b == 64 || b == 128; }
inline int block_log2(int32_t b) { return b == 32 ? 5 : b == 64 ? 6 : 7; }
// Dimensions are kept below 2^24 so that every index fits an int32 after
// division by the block size and element offsets fit 48 bits.
// Rows of dgamma | dbeta partial sums that the first kernel of LayerNorm backward leaves in the workspace: one per
// workgroup, which walks over the groups of 32 rows it owns (at most 512 workgroups).
inline int64_t ln_bwd_partial_rows(int64_t N) { return N / 32 < 512 ? N / 32 : 512; }
// Workspace of LayerNorm backward: the partial rows (dgamma | dbeta, 2 C floats each), and behind them the two row means
// of every row that the first kernel hands to the second (one pair per range of 2048 columns).
inline size_t ln_bwd_workspace_bytes(int64_t N, int64_t C) {
  return (size_t)ln_bwd_partial_rows(N) * 2 * (size_t)C * sizeof(float) + (size_t)N * 2 * sizeof(float) * (size_t)((C + 2047) / 2048);
}
inline bool valid_dim(int64_t d, int32_t block) { return d > 0 && d <= (int64_t(1) << 24) && d % block == 0; }
// A tensor holds at most 2^40 elements (far beyond any device memory): keeps every workgroup count inside 32 bits.
inline bool valid_size(int64_t rows, int64_t cols) { return rows * cols <= (int64_t(1) << 40); }

// Memory that a call reads or writes (p may be null: nothing).  Where an output shares memory with an input, kernels that
// read and write side by side must not take the place of kernels that followed each other.
struct MemRange {
  const void* p;
  int64_t bytes;
};
template <int N, int M>
inline bool any_overlap(const MemRange (&a)[N], const MemRange (&b)[M]) {
  for (const MemRange& x : a)
    for (const MemRange& y : b) {
      const uintptr_t px = reinterpret_cast<uintptr_t>(x.p), py = reinterpret_cast<uintptr_t>(y.p);
      if (px && py && px < py + (uintptr_t)y.bytes && py < px + (uintptr_t)x.bytes) return true;
    }
  return false;
}

// -------------------------------------------------------------- device side
// The kernels that tile a matrix in two dimensions are launched as a one-dimensional grid, column group fastest:
// the y and z dimensions of a grid stop at 65535, which a tensor of 2^24 rows exceeds.
struct TileIndex {
  int x, y;  // column group, row group
};
__device__ __forceinline__ TileIndex tile_of_workgroup(int column_groups, unsigned first = 0) {   // first: workgroups before the tiles
  const unsigned i = blockIdx.x - first;
  TileIndex t;
  t.x = (int)(i % (unsigned)column_groups);
  t.y = (int)(i / (unsigned)column_groups);
  return t;
}
// host side: workgroups of such a launch
inline unsigned tile_grid(int64_t column_groups, int64_t row_groups) { return (unsigned)(column_groups * row_groups); }

// Cross-lane exchange for butterfly reductions without LDS traffic: the value of lane (id ^ 2^BIT) for every lane.
// Bits 0..3 are DPP moves inside a row of 16 lanes (quad permutes, half-row mirror, row rotate by 8); bits 4 and 5
// use the row / half-wave swap instructions of gfx950.  BIT 2 (half-row mirror, lane i <-> 7 - i) equals
// "xor 4" only when the four lanes of every quad already hold the same value, i.e. after the steps for bits 0
// and 1 -- every reduction below that contains bit 2 also contains bits 0 and 1 and takes them first.
// Every lane of the wave must be active.
template <int BIT>
__device__ __forceinline__ int lane_xor_i32(int v) {
  if constexpr (BIT == 0) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false);        // quad_perm [1,0,3,2]
  else if constexpr (BIT == 1) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
  else if constexpr (BIT == 2) return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);  // row_half_mirror
  else if constexpr (BIT == 3) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false);  // row_ror:8
  else if constexpr (BIT == 4) {
    // odd rows of the first operand <-> even rows of the second: (r0 r0 r2 r2) and (r1 r1 r3 r3)
    auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return ((__lane_id() >> 4) & 1) ? (int)p[0] : (int)p[1];
  } else {
    // upper half of the first operand <-> lower half of the second: (lo lo) and (hi hi)
    auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (__lane_id() >> 5) ? (int)p[0] : (int)p[1];
  }
}
template <int BIT>
__device__ __forceinline__ float lane_xor_f32(float v) {
  return __builtin_bit_cast(float, lane_xor_i32<BIT>(__builtin_bit_cast(int, v)));
}
template <int BIT>
__device__ __forceinline__ double lane_xor_f64(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)lane_xor_i32<BIT>((int)(b & 0xffffffffll)), hi = (unsigned)lane_xor_i32<BIT>((int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)lo);
}

template <int MASK, int BIT = 0, class T, class Op, class Xor>
__device__ __forceinline__ T wave_group_reduce(T v, Op op, Xor lane_xor) {
  static_assert(!(MASK & 4) || (MASK & 3) == 3, "the step for bit 2 needs bits 0 and 1 reduced first");
  if constexpr (BIT < 6) {
    if constexpr ((MASK >> BIT) & 1) v = op(v, lane_xor(v, std::integral_constant<int, BIT>()));
    return wave_group_reduce<MASK, BIT + 1>(v, op, lane_xor);
  } else {
    return v;
  }
}

// Max / sum over the lanes whose ids differ only in the bits of MASK (butterfly; every lane of the wave must be
// active).  The summation order is fixed, so results are bit-stable.
template <int MASK>
__device__ __forceinline__ float wave_group_max(float v) {
  return wave_group_reduce<MASK>(v, [](float a, float b) { return fmaxf(a, b); },
                                 [](float x, auto bit) { return lane_xor_f32<decltype(bit)::value>(x); });
}

template <int MASK>
__device__ __forceinline__ float wave_group_sum(float v) {
  return wave_group_reduce<MASK>(v, [](float a, float b) { return a + b; },
                                 [](float x, auto bit) { return lane_xor_f32<decltype(bit)::value>(x); });
}

template <int MASK>
__device__ __forceinline__ double wave_group_sum_f64(double v) {
  return wave_group_reduce<MASK>(v, [](double a, double b) { return a + b; },
                                 [](double x, auto bit) { return lane_xor_f64<decltype(bit)::value>(x); });
}

// Max-abs of 16 values folded into m: eight v_max3_f32 with absolute-value modifiers (the compiler's fmaxf
// quiets each operand with an extra instruction first).
__device__ __forceinline__ float amax16(float m, const float (&y)[16]) {
#pragma unroll
  for (int e = 0; e < 16; e += 2) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(y[e]), "v"(y[e + 1]));
  return m;
}

// The maxima over all lanes of N = 1, 2 or 4 values (none negative) at once: lane l ends with that of value lane_value<N>(l),
// lane value_lane<N>(k) with that of value k.  A swap of half waves or rows between two values and one maximum do a step for
// both, so that four values take 17 instructions where a butterfly each takes 80, and what follows from a maximum (Eq. 1's
// scale, about 30 instructions) is computed once for all of them, each row of lanes for its own.
template <int N>
__device__ __forceinline__ float wave_max_of(const float (&m)[N]) {
  static_assert(N == 1 || N == 2 || N == 4, "halves and rows of a wave");
  // (the swaps read what inline assembly may just have written, which they have to keep two wait states away from)
  const auto larger = [](auto p) __attribute__((always_inline)) {
    float r;
    asm("v_max_f32 %0, %1, %2\n\ts_nop 1" : "=v"(r) : "v"((int)p[0]), "v"((int)p[1]));
    return r;
  };
  const auto bits = [](float v) __attribute__((always_inline)) { return __builtin_bit_cast(int, v); };
  float v[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    v[k] = m[k];
    asm("s_nop 1" : "+v"(v[k]));
  }
  const float a = larger(__builtin_amdgcn_permlane32_swap(bits(v[0]), bits(v[N > 1 ? 1 : 0]), false, false));
  const float b = N == 4 ? larger(__builtin_amdgcn_permlane32_swap(bits(v[N - 2]), bits(v[N - 1]), false, false)) : a;
  float r = larger(__builtin_amdgcn_permlane16_swap(bits(a), bits(b), false, false));
#define JF_ROW_STEP(CTRL) r = __builtin_fmaxf(r, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(bits(r), CTRL, 0xf, 0xf, false)))
  JF_ROW_STEP(0xB1);    // as lane_xor_i32
  JF_ROW_STEP(0x4E);
  JF_ROW_STEP(0x141);
  JF_ROW_STEP(0x128);
#undef JF_ROW_STEP
  return r;
}
template <int N>
__device__ __forceinline__ int lane_value(int lane) { return N == 1 ? 0 : N == 2 ? lane >> 5 : (lane >> 5) | ((lane >> 3) & 2); }
template <int N>
constexpr int value_lane(int k) { return N == 1 ? 0 : 32 * (k & 1) + 16 * (k >> 1); }
// a double from a lane that is the same for all
__device__ __forceinline__ double read_lane_f64(double v, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, lane), hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

constexpr unsigned kLdsBytes = 160 * 1024;   // of a compute unit
typedef __attribute__((address_space(3))) void* lds_ptr;
// One direct-to-LDS load of 16 bytes per lane: lane l's bytes from ubase + voff go to LDS address lds + 16*l.
// Written out because the compiler only selects the 64-bit per-lane address form for the builtin; the form with
// a scalar base and a 32-bit vector offset needs no address arithmetic on the vector ALU.  M0 carries the LDS
// address and needs one wait state before the load reads it.  The load counts in vmcnt like any other; the
// callers wait for it with s_waitcnt before the stage barrier.
// Every direct-to-LDS load of a kernel goes through these helpers, so the compiler itself never uses M0.
__device__ __forceinline__ uint32_t lds_address(const int8_t* lds_tile, int lds_byte) {
  // the tile's LDS address is taken before the byte offset is added: a cast of the sum would carry a null check
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr)(lds_tile) + (uint32_t)lds_byte);
}
__device__ __forceinline__ void load_lds_16(const int8_t* ubase, uint32_t voff, const int8_t* lds_tile, int lds_byte) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(ubase), "s"(lds_address(lds_tile, lds_byte))
               : "memory", "m0");
}
// the same with 4 bytes per lane (lane l's to LDS address lds + 4*l), in that form and with a full 64-bit address per lane
__device__ __forceinline__ void load_lds_4(const void* ubase, uint32_t voff, const int8_t* lds_tile, int lds_byte) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :
               : "v"(voff), "s"(ubase), "s"(lds_address(lds_tile, lds_byte))
               : "memory", "m0");
}
__device__ __forceinline__ void load_lds_4_vaddr(const void* vaddr, const int8_t* lds_tile, int lds_byte) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
               :
               : "v"(vaddr), "s"(lds_address(lds_tile, lds_byte))
               : "memory", "m0");
}
// Kernel arguments.  The first 14 dwords are in registers when the waves start (the build's argument preload); what stands behind them costs
// a trip to memory, 0.3 us in front of a workgroup's first request if the kernel simply has it as a parameter, because the compiler
// reads and awaits parameters at the beginning.  So kernels of a few microseconds have first what their first loads need, and
// read the others where this is called, behind those loads.  ARGS: the argument segment, that is the kernel's parameters in order.
template <class ARGS>
__device__ __forceinline__ const __attribute__((address_space(4))) ARGS* kernel_arguments_from_here() {
  auto p = (const __attribute__((address_space(4))) ARGS*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}
// What such a structure says of its kernel, checked where the kernel is launched: that parameter I is a T that stands `at` bytes into the segment,
// and that the parameters up to I are among those that are preloaded.
constexpr size_t kPreloadedBytes = 14 * 4;
template <class KERNEL>
struct KernelParameters;
template <class... T>
struct KernelParameters<void (*)(T...)> {
  static constexpr size_t end(size_t index, size_t* begin = nullptr) {
    constexpr size_t size[] = {sizeof(T)...}, align[] = {alignof(T)...};
    size_t at = 0;
    for (size_t i = 0; i <= index; ++i) {
      at = (at + align[i] - 1) / align[i] * align[i];
      if (begin) *begin = at;
      at += size[i];
    }
    return at;
  }
  static constexpr size_t begin(size_t index) {
    size_t at = 0;
    end(index, &at);
    return at;
  }
  template <size_t I, class U>
  static constexpr bool stands_at(size_t at) { return std::is_same_v<std::tuple_element_t<I, std::tuple<T...>>, U> && begin(I) == at; }
  template <size_t I>
  static constexpr bool preloaded() { return end(I) <= kPreloadedBytes; }
};
// A pointer that is the same for all lanes, moved to scalar registers for good.
template <class T>
__device__ __forceinline__ T* uniform_pointer(T* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T*)(((uint64_t)hi << 32) | lo);
}

// Results are written through (sc1: agent scope).  Each XCD's L2 is private, so whatever a kernel leaves dirty in it has to
// be written back before the next kernel may start, 1-2 us after a kernel of 10-60 MB; written through, the lines go out
// while the kernel still runs and stay readable in L2 and in the memory-side cache.  Non-temporal stores do the first but
// not the second, which costs the next kernel of a small step more than it saves (MLP step 1152 x 4352 -> 896 at block 128:
// write-back 104, non-temporal 123, write-through 102 us; 4096 x 768 -> 3072: 138, 132, 132; residual path 8192 x 1280: 56,
// 54, 52; GELU 4096 x 3072: 17.1, 15.1, 14.2).  A large result has to be stored in
// whole lines per wave, because a line written through in pieces goes to memory piece by piece (the FP16 hand-over at
// 8192 x 5120 in 16-byte pieces: 87 instead of 71 us); store_part is for what cannot be.
// (Stores the compiler knows: it has to keep the two wait states between a 16-byte store and the next write of its data.)
template <class T>
__device__ __forceinline__ void store_out(void* p, T v) {
  static_assert(sizeof(T) == 16 || sizeof(T) == 8 || sizeof(T) == 4, "one store instruction");
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  if constexpr (sizeof(T) == 16)
    __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) v4u*)p, __builtin_bit_cast(v4u, v), "agent");
  else if constexpr (sizeof(T) == 8)
    __hip_atomic_store((__attribute__((address_space(1))) unsigned long long*)p, __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    __hip_atomic_store((__attribute__((address_space(1))) unsigned*)p, __builtin_bit_cast(unsigned, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_out(void* p, const uint4& v) {
  store_out(p, v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w});
}
// How the operators that run at the speed of memory store a result of `rows` rows of `row_bytes` bytes: chosen by the
// launcher, a template argument of the kernels (a branch in the kernel costs the large tensors 2-3 %).
// Rows that are no multiple of a line share lines between waves, and a result beyond the last-level cache then pays for
// every piece: written back from 32 MB on.  Whole lines that no cache will hold for the reader are streamed from 64 MB on.
// Through / stream / back, block 32, operands from memory (us):
//   1048576 x 768, whole lines   Add 451 / 433 / 452, GELU backward 451 / 436 / 452, Dropout 301 / 286 / 304, LayerNorm 310 /
//                                311 / 315, FP16 quantizer 412 / 402 / 429, FP16 dequantizer 407 / 392 / 411
//   98304 x 768, whole lines     Add 42.5 / 41.0 / 42.6, GELU 29.2 / 28.5 / 30.4, LayerNorm 34.2 / 31.3 / 34.9, backward 60.2 / 58.0 /
//                                62.0, FP32 quantizer 70.1 / 66.6 / 69.5, FP16 dequantizer 39.6 / 37.4 / 40.5
//   199680 x 1504, shared lines  Add 223 / 184 / 180, GELU 161 / 139 / 121, LayerNorm 174 / 154 / 126, backward 254 / 229 / 215,
//                                quantizers and dequantizer equal within 3 %
//   16384 x 1280, whole lines    GELU 9.9 / 10.2 / 11.5, LayerNorm 12.2 / 12.9 / 14.1, FP16 quantizer 10.8 / 11.6 / 12.6
// (Between the bounds, 37 to 68 MB, streaming is 5-15 % faster still for an operator by itself -- LayerNorm 65536 x 768
// 25.3 / 22.2 / 25.5, 24576 x 1504 21.8 / 19.8 / 20.8 -- but takes the result out of the cache that its reader finds it in.)
// The products always write through: their results make up too little of their time for the rule to matter (forward 32768 x
// 768 -> 3104, 101 MB of shared lines, 181 / 182 / 184; 16384 x 4096 -> 4096 485 / 483 / 487).
enum StorePolicy { kStoreThrough, kStoreStream, kStoreBack };
inline StorePolicy store_policy(int64_t rows, int64_t row_bytes) {
  const int64_t bytes = rows * row_bytes;
  if (row_bytes % 128) return bytes >= (32 << 20) ? kStoreBack : kStoreThrough;
  return bytes >= (64 << 20) ? kStoreStream : kStoreThrough;
}
// f(integral_constant<StorePolicy, P>) for the policy of a result
template <class F>
inline void with_store_policy(int64_t rows, int64_t row_bytes, F&& f) {
  const StorePolicy p = store_policy(rows, row_bytes);
  if (p == kStoreThrough) f(std::integral_constant<StorePolicy, kStoreThrough>());
  else if (p == kStoreStream) f(std::integral_constant<StorePolicy, kStoreStream>());
  else f(std::integral_constant<StorePolicy, kStoreBack>());
}
template <StorePolicy P, class T>
__device__ __forceinline__ void store_as(void* p, const T& v) {
  if constexpr (P == kStoreThrough) {
    store_out(p, v);
  } else if constexpr (P == kStoreStream) {
    typedef int many __attribute__((ext_vector_type(sizeof(T) / 4)));
    typedef typename std::conditional<sizeof(T) == 4, int, many>::type vec;
    __builtin_nontemporal_store(__builtin_bit_cast(vec, v), (__attribute__((address_space(1))) vec*)p);
  } else {
    *static_cast<T*>(p) = v;
  }
}
template <class T>
__device__ __forceinline__ void store_part(void* p, T v) { *static_cast<T*>(p) = v; }
// A block's scale beside codes of policy P.  Streamed, the 4 to 16 bytes that a wave has of a grid go to memory by
// themselves, which costs up to 5 % at block 128; written back they are put together in L2 (98304 x 768 at block 128,
// streamed and back: Add 47.5, 45.0 us, FP16 quantizer 48.1, 45.9, LayerNorm backward 84.8, 83.3; 262144 x 768 1-2 %; at
// block 32 and 64 equal within 1 %).  Small grids are written through like their codes (GELU 512 x 768: 3.9 us, written
// back 4.0).
template <StorePolicy P>
__device__ __forceinline__ void store_scale(void* p, float v) {
  if constexpr (P == kStoreStream) store_part(p, v);
  else store_as<P>(p, v);
}

// Eq. 1 scale of a block from its max-abs: one IEEE FP32 division; 0 for an all-zero block.  `inv` is the
// reciprocal of the scale in double precision (0 for an all-zero block, so that every code becomes 0): the
// hardware estimate refined by two Newton steps, relative error below 2^-50.  The double reciprocal exists for
// every FP32 scale, subnormal ones included.
__device__ __forceinline__ void block_scale(float amax, float& scale, double& inv) {
  scale = amax / 127.0f;
  const double s = (double)scale;
  double r = __builtin_amdgcn_rcp(s);
  r = __builtin_fma(__builtin_fma(-s, r, 1.0), r, r);
  r = __builtin_fma(__builtin_fma(-s, r, 1.0), r, r);
  inv = scale > 0.0f ? r : 0.0;
}

// round-half-even(x / scale) of the EXACT quotient of the two FP32 numbers (Eq. 1), as an integer in the low
// byte of the result.  A quotient of two FP32 numbers is either exactly k + 1/2 or at least 2^-26 away from it,
// so it suffices to know it to better than that, which x * inv in double does (error below 127.5 * 2^-50):
//   t1 = fma(x, inv, 1.5 * 2^20)    lies in one binade with ulp 2^-32: everything within 2^-33 of k + 1/2 -- only
//                                   exact ties are -- lands exactly on the tie, everything else stays on its side;
//   t  = t1 + (1.5 * 2^52 - 1.5 * 2^20)   rounds to an integer, the exact tie to even (1.5 * 2^52 is even), and
//                                   leaves it in the low mantissa bits (two's complement modulo 256 in bits 0..7).
// An FP32 product x * (1/scale) cannot do this: its error of up to 7.6e-6 decides every tie and near-tie at
// random, and tensors whose blocks keep their scale through an operator consist of little else.
__device__ __forceinline__ uint32_t code_bits(float x, double inv) {
  const double t1 = __builtin_fma((double)x, inv, 1572864.0);
  const double t = t1 + (6755399441055744.0 - 1572864.0);
  return (uint32_t)__builtin_bit_cast(unsigned long long, t);
}

// Pack the low bytes of four code_bits() results into one dword, a0 lowest.
__device__ __forceinline__ uint32_t pack_codes(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
  uint32_t lo = __builtin_amdgcn_perm(a1, a0, 0x0c0c0400u);  // [a0.b0, a1.b0, 0, 0]
  uint32_t hi = __builtin_amdgcn_perm(a3, a2, 0x04000c0cu);  // [0, 0, a2.b0, a3.b0]
  return lo | hi;
}

__device__ __forceinline__ uint32_t quantize4(float x0, float x1, float x2, float x3, double inv) {
  return pack_codes(code_bits(x0, inv), code_bits(x1, inv), code_bits(x2, inv), code_bits(x3, inv));
}

// Signed byte k (0..3) of a packed dword as float.
__device__ __forceinline__ float byte_to_float(uint32_t packed, int k) {
  return (float)((int32_t)(packed << (24 - 8 * k)) >> 24);
}

}  // namespace jf
