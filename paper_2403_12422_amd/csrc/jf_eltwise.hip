// INT8-in / INT8-out GELU (forward and backward), Add and Dropout (Sec. 6, Alg. 2, App. A).
//
// These kernels move 2-3 bytes per element, so at HBM speed a SIMD has 50-60 cycles per element, of which Eq. 1's exact
// rounding takes 14.  What keeps them inside that budget:
//   * GELU: within one quantization block the input takes at most 255 values (code * block scale), so GELU (or its
//     derivative) is tabulated once per block in LDS and every element is a table lookup indexed by its code byte -- the
//     dequantize step of Alg. 2 and the erf evaluation collapse into it;
//   * one wave per strip of 32 x 128, 64 elements of one block per lane, see jf_rowops.hpp; at block size 32 no barrier.  A few
//     million elements give a SIMD a wave or two, whose time is that serial chain: there waves of 16 rows halve it.
#include "jf_rowops.hpp"

namespace jf {

// ------------------------------------------------------------------------------------------------
// One table of GELU (or its derivative) at the 255 values code * sx of a block, indexed by the code byte taken as
// unsigned: lane l evaluates codes l and l + 64 and, by symmetry, -l and -(l + 64).  Both functions are written in
// terms of the upper tail Q(a) = Phi(-a), a >= 0 (App. A):
//   GELU(x) = x Phi(x):  f(a) = a - a Q(a),  f(-a) = -a Q(a);
//   GELU'(x) = Phi(x) + x phi(x):  f(a) = 1 - Q(a) + a phi(a),  f(-a) = Q(a) - a phi(a),  phi(a) = exp(-a^2/2) / sqrt(2 pi).
//   Q(a) = t P(t) exp(-a^2/2),  t = 1 / (1 + a / sqrt(8)),  P of degree 8 fitted by weighted least squares on Chebyshev
//   nodes to erfcx(a / sqrt 2) / (2 t) for 0 <= a <= 13.4 (relative error 5e-8; evaluated in FP32: 4e-7).
// exp(-a^2/2) = 2^H (1 + r ln 2) with H = fl(-a^2 log2(e)/2) and r the exact remainder (product residuals by FMA),
// so that the FP32 rounding of an exponent of size a^2 does not cost log2(a^2) bits: Q keeps a relative error of
// about 1e-6 into the far tail, where a block that lies entirely there takes its scale from.
template <bool BWD>
__device__ __forceinline__ void gelu_table_entries(float a, float& pos, float& neg) {
  const float ac = fminf(a, 40.0f);                       // Q(40) = 0 in FP32; keeps a^2 finite
  const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(ac, 0.35355339059327373f, 1.0f));
  float p = -2.9970746985e-02f;
  p = __builtin_fmaf(p, t, 1.4432375881e-01f);
  p = __builtin_fmaf(p, t, -2.4760739076e-01f);
  p = __builtin_fmaf(p, t, 1.4335782902e-01f);
  p = __builtin_fmaf(p, t, -1.6097390692e-02f);
  p = __builtin_fmaf(p, t, 1.0243339323e-01f);
  p = __builtin_fmaf(p, t, 1.2129997806e-01f);
  p = __builtin_fmaf(p, t, 1.4121892641e-01f);
  p = __builtin_fmaf(p, t, 1.4104161820e-01f);
  const float K = -0.72134752044448170f;                  // -log2(e) / 2
  const float aa = ac * ac;
  const float lo = __builtin_fmaf(ac, ac, -aa);           // a^2 = aa + lo exactly
  const float H = aa * K;
  const float r = __builtin_fmaf(lo, K, __builtin_fmaf(aa, K, -H));
  const float ez = __builtin_amdgcn_exp2f(H) * __builtin_fmaf(r, 0.6931471805599453f, 1.0f);   // exp(-a^2/2)
  const float q = (t * p) * ez;
  if (BWD) {
    const float s = (a * 0.39894228040143268f) * ez;      // a phi(a)
    pos = (1.0f - q) + s;
    neg = q - s;
  } else {
    const float aq = a * q;
    pos = a - aq;
    neg = 0.0f - aq;
  }
}

// Entries of lane `i` of a half table: those of the codes i and -i (i = 64 half + lane).
// code 0: GELU(0) = 0 comes out exactly; GELU'(0) = 1/2 is set, because the fit is only good to 4e-7 there and a
// derivative of 0.49999997 would push every halved gradient code off its rounding tie.  Entry 128 (code -128,
// which no quantizer output holds) is 0.
struct TablePair {
  float pos, neg;
};
template <bool BWD>
__device__ __forceinline__ TablePair gelu_table_pair(float sx, int i) {
  TablePair e;
  gelu_table_entries<BWD>((float)i * sx, e.pos, e.neg);
  if (BWD && i == 0) e.pos = 0.5f;
  if (i == 0) e.neg = 0.0f;
  return e;
}
__device__ __forceinline__ int table_pos(int i) { return i; }
__device__ __forceinline__ int table_neg(int i) { return i == 0 ? 128 : 256 - i; }

// Between LDS accesses of one wave, which LDS serves in program order: keeps the compiler from moving one past the other.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The largest signed code of a lane's 16 P codes.  (Two at a time, each the upper byte of 16 bits: what stands below it does not decide.)
template <int P>
__device__ __forceinline__ int largest_code(const uint4 (&v)[P]) {
  typedef short v2s __attribute__((ext_vector_type(2)));
  v2s m = __builtin_bit_cast(v2s, v[0].x);
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const v2s odd = __builtin_bit_cast(v2s, d == 0 ? v[p].x : d == 1 ? v[p].y : d == 2 ? v[p].z : v[p].w);
      m = __builtin_elementwise_max(__builtin_elementwise_max(m, odd), (v2s)(odd << 8));
    }
  return max(m[0] >> 8, m[1] >> 8);
}
// Of the same codes the smallest that is not below `at`, and the largest below it; above 127 and below -128: there is none.  Differences modulo
// 256 put the codes from `at` up first and those below it last, the next one at the very end.
template <int P>
__device__ __forceinline__ void codes_around(const uint4 (&v)[P], int at, int& from, int& below) {
  typedef unsigned short v2u __attribute__((ext_vector_type(2)));
  const v2u origin = (v2u)(unsigned short)(at << 8);
  v2u first = (v2u)(unsigned short)0xffff, last = (v2u)(unsigned short)0;
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const v2u two = __builtin_bit_cast(v2u, d == 0 ? v[p].x : d == 1 ? v[p].y : d == 2 ? v[p].z : v[p].w);
      const v2u odd = two - origin, even = (v2u)(two << 8) - origin;
      first = __builtin_elementwise_min(__builtin_elementwise_min(first, odd), even);
      last = __builtin_elementwise_max(__builtin_elementwise_max(last, odd), even);
    }
  from = at + (min(first[0], first[1]) >> 8);
  below = at + (max(last[0], last[1]) >> 8) - 256;
}

// GELU forward and backward (BWD: dx = g GELU'(x)) on strips: a table per block and wave, or, with waves of 16 rows, per block of a
// strip, built by the waves that share it.
//
// Forward, a block's results are a function of the code alone, and so are their codes: the table is quantized, 256 entries for the 1024 elements
// of a block, and an element is one byte looked up.  That takes the block's max-abs before the first lookup.  GELU grows with x > 0, and -GELU(-a)
// grows with a up to 0.7518, where it is 0.17, and falls beyond.  So the max-abs is GELU of the largest code if that stands for 0.3 or more, else the
// largest of it and of the two codes next to -0.7518 on either side.  (Between neighbouring codes GELU changes by 4e-5 of itself or more, there too,
// and FP32 evaluates it to 1e-6, so that the order of the codes is that of the table's entries.)  Blocks without an ordinary scale, and those whose
// results are next to none, where that is not so, take FP32 tables, and Eq. 1 for each element.
// (Forward, us, FP32 tables -> quantized, ordinary activations: 32768 x 4096 from memory 51.5 -> 44, 8192 x 5120 from the last-level cache 18 -> 14.5,
// 8192 x 1280 6.0 -> 5.75, 1024 x 1024 3.3 -> 3.15.  Where every block is below -0.3 so that the smaller codes decide: 32768 x 4096 50 -> 48, 8192 x 5120
// 17.4 -> 17, 8192 x 1280 5.75 -> 6.6, 1024 x 1024 3.3 -> 3.4; in 1 % of the blocks 8192 x 1280 6.0 -> 6.0.  With the max-abs found by looking
// FP32 values up first 8192 x 1280 took 13 % longer than without quantized tables.)
template <bool BWD, int B, int WAVES, int RW, StorePolicy SP>
__global__ void __launch_bounds__(64 * WAVES) gelu_kernel(const int8_t* __restrict__ X, const float* __restrict__ SX, const int8_t* __restrict__ G,
                                                         const float* __restrict__ SG, int rows, int cols, int8_t* __restrict__ Y, float* __restrict__ SY) {
  constexpr int NBC = 128 / B;   // blocks of a strip
  constexpr int SHARED = RW < 32 ? Strip<B, WAVES, RW>::BT : 1;   // waves that share a strip's tables
  __shared__ __align__(1024) float s_tabs[WAVES / SHARED][NBC][256];
  __shared__ float s_amax[WAVES][4], s_amax32[WAVES][4];
  const Strip<B, WAVES, RW> t(rows, cols);
  constexpr int P = Strip<B, WAVES, RW>::PASSES, BT = Strip<B, WAVES, RW>::BT;
  if (BT == 1 && !t.inside) return;   // a whole wave; there is no workgroup barrier
  const int64_t pass = (int64_t)8 * cols;
  uint4 px[P], pg[BWD ? P : 1];   // requested first: their latency runs beside the table build
#pragma unroll
  for (int p = 0; p < P; ++p) {
    px[p] = *reinterpret_cast<const uint4*>(X + t.base + p * pass);
    if (BWD) pg[p] = *reinterpret_cast<const uint4*>(G + t.base + p * pass);
  }
  // the strip's block scales are the same for all lanes: scalar loads (the grids are not written by this kernel before the
  // barrier, and at block size 32 by nobody else)
  typedef const __attribute__((address_space(4))) float* const_f32_ptr;
  const const_f32_ptr sx_row = (const_f32_ptr)SX + (int64_t)(t.bi / BT) * t.lc + t.c0 / B;
  const int nblk = min(NBC, t.lc - t.c0 / B);
  // this wave's part of the strip's tables: half tables, in turn with the waves that share them
  constexpr int HALVES = (2 * NBC + SHARED - 1) / SHARED;   // (at block size 128 two of eight waves have one)
  const auto half_of = [&](int u) __attribute__((always_inline)) { return u * SHARED + (SHARED == 1 ? 0 : t.wave % SHARED); };
  const auto code_of = [&](int h) __attribute__((always_inline)) { return t.lane + 64 * (h & 1); };
  TablePair entry[HALVES];
#pragma unroll
  for (int u = 0; u < HALVES; ++u) {
    const int h = half_of(u);
    entry[u] = gelu_table_pair<BWD>(sx_row[min(h / 2, nblk - 1)], code_of(h));
  }
  const int own_table = t.ch / (B / 16);
  const auto tables_built = [&]() __attribute__((always_inline)) {
    if constexpr (SHARED == 1) wave_lds_order();
    else __syncthreads();
  };

  float scale;
  uint4 o[P];
  bool quantized = false;
  if constexpr (!BWD) {
    // ---- the table quantized
    const float sx = sx_row[min(own_table, nblk - 1)];
    const auto result_of = [&](int code) __attribute__((always_inline)) {   // |GELU| of a code's input
      float pos, neg;
      const float a = fabsf((float)code) * sx;
      gelu_table_entries<false>(a, pos, neg);
      return fabsf(code > 0 ? pos : neg);   // (no -0: a scale is 0 or more)
    };
    constexpr float kEnough = 0.3f, kLowest = 0.7517915f, kHuge = 3.0e38f, kLeast = 0x1p-100f;
    int code = max(largest_code(px), 0);   // whose result this lane brings
    float amax = result_of(code);
    bool ordinary = true;
    if (__builtin_expect(__any(!((float)code * sx >= kEnough)), 0)) {
      // Four lanes of a block at a time put their codes together, and each brings the result of one.
      int from, below;
      codes_around(px, -(int)__builtin_amdgcn_fmed3f(kLowest * __builtin_amdgcn_rcpf(sx), 0.0f, 127.0f), from, below);
      const auto over4 = [](int v, auto op) __attribute__((always_inline)) {
        return wave_group_reduce<9>(v, op, [](int x, auto bit) { return lane_xor_i32<decltype(bit)::value>(x); });
      };
      const auto larger = [](int a, int b) { return max(a, b); };
      code = over4(code, larger);
      from = over4(from, [](int a, int b) { return min(a, b); });
      below = over4(below, larger);
      const int turn = t.lane & 9;
      if (turn == 1) code = min(from, 0);
      if (turn == 8) code = below > -128 ? below : 0;   // (code -128 has entry 0)
      ordinary = sx >= 0.0f && 128.0f * sx < kHuge;
      amax = result_of(code);
    }
    // a result beyond kHuge (or infinite, or none) has to stay in the block's maximum, which is refused then
    amax = wave_group_max<56 | (B / 16 - 1)>(ordinary && amax < kHuge ? amax : kHuge);
    float voted = amax;   // where a strip has several waves: a block of the workgroup for each lane, so that all of them come to the same
    if constexpr (BT > 1) {
      if ((t.lane & (56 | (B / 16 - 1))) == 0) s_amax[t.wave][own_table] = amax;
      __syncthreads();
      const int first = min(t.lane / NBC, WAVES / BT - 1) * BT;
      voted = 0.0f;
#pragma unroll
      for (int k = 0; k < BT; ++k) {
        amax = fmaxf(amax, s_amax[t.wave / BT * BT + k][own_table]);
        voted = fmaxf(voted, s_amax[first + k][t.lane % NBC]);
      }
    }
    quantized = !__any(!(voted == 0.0f || (voted >= kLeast && voted < kHuge)));
    if (__builtin_expect(quantized, 1)) {
      double inv;
      block_scale(amax, scale, inv);
      int8_t* const codes = reinterpret_cast<int8_t*>(s_tabs[t.wave / SHARED]);   // 256 of each block
#pragma unroll
      for (int u = 0; u < HALVES; ++u) {
        static_assert(BWD || 2 * NBC % SHARED == 0, "a wave has whole half tables to do");
        const int h = half_of(u), i = code_of(h);
        const double k = read_lane_f64(inv, h / 2 * (B / 16));
        codes[h / 2 * 256 + table_pos(i)] = (int8_t)code_bits(entry[u].pos, k);
        codes[h / 2 * 256 + table_neg(i)] = (int8_t)code_bits(entry[u].neg, k);
      }
      tables_built();
      typedef __attribute__((address_space(3))) uint8_t* lds_u8;
      const uint32_t base = (uint32_t)(uintptr_t)(lds_ptr)(codes) + 256 * own_table;   // a multiple of 256, below 65536
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const uint32_t w[4] = {px[p].x, px[p].y, px[p].z, px[p].w};
        uint32_t r[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          uint32_t c[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) c[e] = *(lds_u8)(uintptr_t)__builtin_amdgcn_perm(w[d], base, 0x0c0c0104u + e);   // the code below the base's second byte
          r[d] = (c[0] | c[1] << 8) | (c[2] | c[3] << 8) << 16;
        }
        o[p] = make_uint4(r[0], r[1], r[2], r[3]);
      }
    }
  }
  if (!quantized) {
    // ---- FP32 tables
#pragma unroll
    for (int u = 0; u < HALVES; ++u) {
      const int h = half_of(u), i = code_of(h);
      if (h >= 2 * NBC) break;
      s_tabs[t.wave / SHARED][h / 2][table_pos(i)] = entry[u].pos;
      s_tabs[t.wave / SHARED][h / 2][table_neg(i)] = entry[u].neg;
    }
    tables_built();
    const float* const tab = s_tabs[t.wave / SHARED][own_table];
    float sg = 0.0f, sg128 = 0.0f;
    if (BWD) {
      sg = SG[t.block_index()];
      sg128 = -128.0f * sg;
    }
    const auto results = [&](int p, float (&y)[16]) __attribute__((always_inline)) {
      const uint32_t w[4] = {px[p].x, px[p].y, px[p].z, px[p].w};
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        y[4 * d + 0] = tab[w[d] & 0xffu];
        y[4 * d + 1] = tab[(w[d] >> 8) & 0xffu];
        y[4 * d + 2] = tab[(w[d] >> 16) & 0xffu];
        y[4 * d + 3] = tab[w[d] >> 24];
      }
      if (BWD) {
        float ug[16];
        unpack16_biased(pg[p], ug);
#pragma unroll
        for (int e = 0; e < 16; ++e) y[e] = __builtin_fmaf(ug[e], sg, sg128) * y[e];
      }
    };
    float m = 0.0f;
    double inv;
    if constexpr (BWD) {
      float y[P][16];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        results(p, y[p]);
        m = amax16(m, y[p]);
      }
      strip_block_scale(m, t, s_amax32, scale, inv);
#pragma unroll
      for (int p = 0; p < P; ++p) o[p] = quantize16(y[p], inv);
    } else {   // looked up twice: kept, the results would take the registers of a wave on every SIMD
      float y[16];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        results(p, y);
        m = amax16(m, y);
        __builtin_amdgcn_sched_barrier(0);
      }
      strip_block_scale(m, t, s_amax32, scale, inv);
#pragma unroll
      for (int p = 0; p < P; ++p) {
        results(p, y);
        o[p] = quantize16(y, inv);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (!t.ok) return;
  if (t.owns_scale()) store_scale<SP>(&SY[t.block_index()], scale);
#pragma unroll
  for (int p = 0; p < P; ++p) store_as<SP>(Y + t.base + p * pass, o[p]);
}

// ------------------------------------------------------------------------------------------------
// Add (App. A): y = x1 + x2 on the dequantized operands, re-quantized per block (Alg. 2), and optionally
// the row partials that App. A's LayerNorm paragraph attaches to this operator: for every row and block
// column, the mean and the sum of squares of y over the block's B columns (stored block-column-major).
// The row partials are 8 bytes per row and block column, a quarter of the codes at B = 32.  They are written back whatever the
// codes' policy, since a wave has whole lines of them at block sizes 64 and 128 only (streamed in pieces, 1048576 x 768 at
// block 32 took 653 us, written through 543, back 472), and each lane stores those of another pass: two or four stores per
// strip for eight of a few lanes each (8192 x 1280 7.6 -> 7.3 us, 1048576 x 768 469 -> 447; at block 128 7.5 -> 7.4, 468 -> 409).
template <int B, int WAVES, int RW, bool PARTIALS, StorePolicy SP>
__global__ void __launch_bounds__(64 * WAVES) add_kernel(const int8_t* __restrict__ X1, const float* __restrict__ S1,
                                                              const int8_t* __restrict__ X2, const float* __restrict__ S2, int rows, int cols,
                                                              int8_t* __restrict__ Y, float* __restrict__ SY, float* __restrict__ row_mean,
                                                              float* __restrict__ row_sumsq) {
  __shared__ float s_amax[WAVES][4];
  const Strip<B, WAVES, RW> t(rows, cols);
  constexpr int P = Strip<B, WAVES, RW>::PASSES;
  if (t.BT == 1 && !t.inside) return;   // a whole wave; there is no workgroup barrier
  const int64_t pass = (int64_t)8 * cols;
  float y[P][16], ps[P], pq[P];
  float m = 0.0f;
  uint4 p1[P], p2[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    p1[p] = *reinterpret_cast<const uint4*>(X1 + t.base + p * pass);
    p2[p] = *reinterpret_cast<const uint4*>(X2 + t.base + p * pass);
  }
  const float s1 = S1[t.block_index()], s2 = S2[t.block_index()];
  const float k = -128.0f * (s1 + s2);  // the unpacked codes carry +128
#pragma unroll
  for (int p = 0; p < P; ++p) {
    float u1[16], u2[16];
    unpack16_biased(p1[p], u1);
    unpack16_biased(p2[p], u2);
#pragma unroll
    for (int e = 0; e < 16; ++e) y[p][e] = __builtin_fmaf(u1[e], s1, __builtin_fmaf(u2[e], s2, k));
    m = amax16(m, y[p]);
    if (PARTIALS) {  // per row and block: mean and sum of squares over the block's columns = B / 16 neighbouring lanes
      ps[p] = pq[p] = 0.0f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        ps[p] += y[p][e];
        pq[p] = __builtin_fmaf(y[p][e], y[p][e], pq[p]);
      }
      ps[p] = wave_group_sum<B / 16 - 1>(ps[p]) * (1.0f / (float)B);
      pq[p] = wave_group_sum<B / 16 - 1>(pq[p]);
    }
  }
  if (PARTIALS && t.ok) {
    // Block-column-major: the 32 rows of the strip are one 128-byte line per block column.  All lanes of a block hold its sums
    // of the four passes; each stores those of another pass.
    float* const mean = row_mean + (int64_t)(t.col / B) * rows + t.bi * RW + t.rsub;
    float* const sumsq = row_sumsq + (int64_t)(t.col / B) * rows + t.bi * RW + t.rsub;
    const auto pick = [](bool second, float a, float b) { return second ? b : a; };   // (by value: of references it would be an address)
    const int k = t.ch & (B / 16 - 1), p = k & (P - 1);
    const auto of_pass = [&](const float(&v)[P]) {
      if constexpr (P == 4) return pick(p & 2, pick(p & 1, v[0], v[1]), pick(p & 1, v[2], v[3]));
      else return pick(p, v[0], v[1]);
    };
    if constexpr (B == 32) {
#pragma unroll
      for (int i = 0; i < P; i += 2) {
        store_part(&mean[8 * (i + k)], pick(k, ps[i], ps[i + 1]));
        store_part(&sumsq[8 * (i + k)], pick(k, pq[i], pq[i + 1]));
      }
    } else if constexpr (B / 16 < 2 * P) {
      store_part(&mean[8 * p], of_pass(ps));
      store_part(&sumsq[8 * p], of_pass(pq));
    } else if (k < 2 * P) {
      store_part((k < P ? mean : sumsq) + 8 * p, pick(k < P, of_pass(pq), of_pass(ps)));
    }
  }
  float scale;
  double inv;
  strip_block_scale(m, t, s_amax, scale, inv);
  if (!t.ok) return;
  if (t.owns_scale()) store_scale<SP>(&SY[t.block_index()], scale);
#pragma unroll
  for (int p = 0; p < P; ++p) store_as<SP>(Y + t.base + p * pass, quantize16(y[p], inv));
}

// ------------------------------------------------------------------------------------------------
// The codes of a packed dword whose keep bits are set, the four bits of `nibble`, which is less than 16; 0 for the others.  The
// multiplication puts bit j at bit 8 j + 2 (and copies elsewhere), where it makes the byte selector j + 4, byte j of `codes`, instead of
// j, a byte of zero.
__device__ __forceinline__ uint32_t kept_codes(uint32_t codes, uint32_t nibble) {
  const uint32_t at = __umul24(nibble, 0x00810204u);
  uint32_t select;   // (at & mask) | (identity & ~mask): the compiler has no single instruction of its own for it here
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(select) : "s"(0x04040404u), "v"(at), "v"(0x03020100u));
  return __builtin_amdgcn_perm(codes, 0u, select);
}

// Dropout (App. A): y = x o m / (1 - p) on the dequantized input, re-quantized per block; the keep mask m is an input, packed 8
// columns per byte (bit c % 8 of byte c / 8 of a row).  The backward pass is the same operator on the upstream gradient.
// Dropped codes are cleared in the packed dwords (a code of 0 dequantizes to exactly 0), so the mask costs one instruction per element.
//
// All elements of a block are y = fl(c k) for one k and a code c, so that Eq. 1 is a function of c and the largest |c| left, m: its
// quotient is 127 c / m but for relative 2^-22.  127 c / m is at least 1 / (2 m) away from a tie, or is one, which happens at c = +-m / 2
// only (127 is prime).  So one FP32 FMA with 127 / m rounds every other code; and at m / 2, where fl(m k) = 2 fl(m k / 2), it is beyond 63.5 or
// not as the scale fl(amax / 127) lies below amax / 127 or above it: the factor is moved by 2^-20 of itself to that side (a scale that is
// amax / 127 exactly makes a tie, which goes to 64).  The moved factor takes no other code past a tie: 127 * 2^-20 < 1 / 256.
// That holds while k and amax are no subnormals and finite; a wave with other blocks takes the general rounding, but for blocks of k = 0 (padding,
// dead channels), whose codes are all 0.
// (Vector instructions per element 8.9 -> 5.8.  8192 x 1280 from the last-level cache 5.0 -> 4.0 us, from memory 6.6 -> 6.25, at block 64 and 128 6.6 -> 6.3
// and 7.0 -> 6.6; 16384 x 2560 19.3 -> 18.2; 262144 x 3072 307, as before: the memory.  Residual path of 8192 x 1280 46.8 -> 45.6.)
template <int B, int WAVES, int RW, StorePolicy SP>
__global__ void __launch_bounds__(64 * WAVES) dropout_kernel(const int8_t* __restrict__ X, const float* __restrict__ SX,
                                                                  const uint8_t* __restrict__ mask, float keep_scale, int rows, int cols,
                                                                  int8_t* __restrict__ Y, float* __restrict__ SY) {
  __shared__ float s_amax[WAVES][4];
  const Strip<B, WAVES, RW> t(rows, cols);
  constexpr int P = Strip<B, WAVES, RW>::PASSES;
  if (t.BT == 1 && !t.inside) return;   // a whole wave; there is no workgroup barrier
  const int64_t pass = (int64_t)8 * cols;
  float m = 0.0f;
  uint4 px[P];
  uint32_t bits[P];
  const int64_t mbase = t.base >> 3;   // row * (cols / 8) + column / 8: cols is a multiple of 32, the column of 16
#pragma unroll
  for (int p = 0; p < P; ++p) {
    px[p] = *reinterpret_cast<const uint4*>(X + t.base + p * pass);
    bits[p] = *reinterpret_cast<const uint16_t*>(mask + mbase + (int64_t)p * cols);   // 8 rows further: 8 * cols / 8 bytes
  }
  const float k = SX[t.block_index()] * keep_scale;
  float c[P][16];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint32_t w[4] = {kept_codes(px[p].x, bits[p] & 15u), kept_codes(px[p].y, (bits[p] >> 4) & 15u), kept_codes(px[p].z, (bits[p] >> 8) & 15u),
                           kept_codes(px[p].w, bits[p] >> 12)};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
      for (int e = 0; e < 4; ++e) c[p][4 * d + e] = (float)(int8_t)(w[d] >> 8 * e);
    }
    m = amax16(m, c[p]);
  }
  m = strip_block_max(m, t, s_amax);
  const float k128 = -128.0f * k;
  // The largest |c k|, exactly 0 or of the code with it; of a k that is not finite what the general rounding below makes of it, without an exchange.
  const float amax = fmaxf(fabsf(__builtin_fmaf(m + 128.0f, k, k128)), 0.0f);
  uint4 o[P];
  float scale;
  if (__builtin_expect(!__any(!(k == 0.0f || (k >= 0x1p-100f && k <= 0x1p100f))), 1)) {
    scale = amax / 127.0f;
    const float over = __builtin_fmaf(scale, 127.0f, -amax);   // exact in sign: of scale - amax / 127
    const float f = amax > 0.0f ? 127.0f * __builtin_amdgcn_rcpf(m) * (over > 0.0f ? 1.0f - 0x1p-20f : 1.0f + 0x1p-20f) : 0.0f;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      uint32_t r[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) r[e] = __builtin_bit_cast(uint32_t, __builtin_fmaf(c[p][e], f, 12582912.0f));   // 1.5 * 2^23: an integer, in the low bits
      o[p] = make_uint4(pack_codes(r[0], r[1], r[2], r[3]), pack_codes(r[4], r[5], r[6], r[7]), pack_codes(r[8], r[9], r[10], r[11]),
                        pack_codes(r[12], r[13], r[14], r[15]));
    }
  } else {
    double inv;
    block_scale(amax, scale, inv);
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
      for (int e = 0; e < 16; ++e) c[p][e] = __builtin_fmaf(c[p][e] + 128.0f, k, k128);
      o[p] = quantize16(c[p], inv);
    }
  }
  if (!t.ok) return;
  if (t.owns_scale()) store_scale<SP>(&SY[t.block_index()], scale);
#pragma unroll
  for (int p = 0; p < P; ++p) store_as<SP>(Y + t.base + p * pass, o[p]);
}

// ------------------------------------------------------------------------------------------------ host
// Whether an operator takes waves of 16 rows (for results that are written through).  Small tensors give a SIMD a wave or two, and a wave of
// 16 rows has half the serial chain.  From a few million elements on it matters how the waves come out on 1024 SIMDs: 32-row waves fill
// rounds of 4 M elements, half waves round a rest less up, and cost twice the scales, reductions and exchanges.  The lines lie where the
// gain ends in the paths of a training step, or before, where an operator alone on operands from memory begins to lose; all figures are in
// profiles/strip_heights.txt.  32 -> 16 rows in us, alone from memory | from the last-level cache | in its path:
//   GELU forward, block 32   1 M elements 3.7 -> 3.1 | 3.7 -> 3.1   14 M 8.35 -> 8.0 | 6.7 -> 6.85 | 132.8 -> 131.7   15 M 8.75 -> 9.75 | 6.8 -> 7.45 | 137.1 -> 136.0
//     block 64   11 M 6.3 -> 5.9 | 5.1 -> 5.1 | 102.6 -> 100.2   12 M 7.2 -> 8.0 | 5.25 -> 5.2 | 104.4 -> 102.4      block 128: eight waves to a table, nowhere
//     rows that share lines   27 M 17.3 -> 16.9 | 10.8 -> 12.1 | 250.7 -> 249.0   31 M 18.4 -> 19.1 | 13.15 -> 13.95 | 226.9 -> 225.6
//   GELU backward, block 32   13 M 11.55 -> 11.0 | 8.15 -> 7.95 | 131.5 -> 129.8   14 M 11.9 -> 11.1 | 8.3 -> 8.1 | 135.0 -> 135.1   16 M 12.8 -> 12.7 | 8.45 -> 9.05 |
//     140.2 -> 141.2; rows that share lines 17 M 16.85 -> 16.45 | 11.65 -> 13.0 | 166.5 -> 166.3   block 64   11 M 9.6 -> 9.5 | 6.85 -> 6.45 | 102.2 -> 100.3   12 M
//     9.85 -> 11.1 | 7.0 -> 6.5 | 103.4 -> 104.6
//   Add, alone 1 M 3.8 -> 3.3, block 64 and 128 3.9 -> 3.2 and 4.1 -> 3.6; in the residual path at block 32 10 M 53.7 -> 53.8, 12 M 63.8 -> 63.4, 16 M
//     76.5 -> 75.7, 20 M 86.7 -> 86.0, by up to 2 % the one or the other way from width to width; block 128 16 M 83.8 -> 82.7
//   Dropout, block 32   1 M 2.7 -> 2.65 | 2.7 -> 2.5 | 23.9 -> 22.8   4 M 3.6 -> 3.7 | 3.05 -> 3.0 | 30.5 -> 30.0   8 M, path only, 38.3 -> 39.3
static bool low_gelu(bool backward, int block, int64_t rows, int64_t cols) {
  const bool shared = cols % 128;   // rows that share lines
  const int most = backward ? (block == 128 ? 16 : block == 64 ? (shared ? 12 : 11) : shared ? 18 : 13) : block == 64 ? 11 : 14;   // in 2^20 elements
  return (!backward && shared) || rows * cols <= int64_t(most) << 20;
}
static bool low_add(int block, int64_t rows, int64_t cols) { return rows * cols <= (block == 128 ? 32 : block == 64 ? 12 : 11) << 20; }
static bool low_dropout(int64_t rows, int64_t cols) { return rows * cols <= 4 << 20; }

template <bool BWD>
static void launch_gelu(int block, const int8_t* X, const float* SX, const int8_t* G, const float* SG, int rows, int cols, int8_t* Y, float* SY,
                        hipStream_t st) {
  with_instance<BWD>(block, rows, cols, low_gelu(BWD, block, rows, cols), [&](auto b, auto w, auto r, auto sp) {
    constexpr int B = decltype(b)::value, WAVES = decltype(w)::value, RW = decltype(r)::value;
    constexpr StorePolicy SP = decltype(sp)::value;
    hipLaunchKernelGGL((gelu_kernel<BWD, B, WAVES, RW, SP>), (strip_grid<B, WAVES, RW>(rows, cols)), dim3(64 * WAVES), 0, st, X, SX, G, SG, rows, cols, Y, SY);
  });
}

}  // namespace jf

extern "C" int32_t jf_gelu_q(const int8_t* X, const float* SX, int64_t N, int64_t C, int32_t block, int8_t* Y,
                             float* SY, void* stream) {
  using namespace jf;
  int32_t rc = check_eltwise(X, SX, Y, SY, N, C, block);
  if (rc != JF_OK) return rc;
  launch_gelu<false>(block, X, SX, nullptr, nullptr, (int)N, (int)C, Y, SY, reinterpret_cast<hipStream_t>(stream));
  return launch_status();
}

extern "C" int32_t jf_gelu_q_bwd(const int8_t* dY, const float* SdY, const int8_t* X, const float* SX, int64_t N,
                                 int64_t C, int32_t block, int8_t* dX, float* SdX, void* stream) {
  using namespace jf;
  int32_t rc = check_eltwise(X, SX, dX, SdX, N, C, block);
  if (rc != JF_OK) return rc;
  if (!dY || !SdY) return JF_ERR_NULL;
  if (!aligned16(dY) || !aligned4(SdY)) return JF_ERR_ALIGN;
  launch_gelu<true>(block, X, SX, dY, SdY, (int)N, (int)C, dX, SdX, reinterpret_cast<hipStream_t>(stream));
  return launch_status();
}

extern "C" int32_t jf_dropout_q(const int8_t* X, const float* SX, const uint8_t* mask_bits, float p, int64_t N, int64_t C,
                                int32_t block, int8_t* Y, float* SY, void* stream) {
  using namespace jf;
  int32_t rc = check_eltwise(X, SX, Y, SY, N, C, block);
  if (rc != JF_OK) return rc;
  if (!mask_bits) return JF_ERR_NULL;
  if (!(p >= 0.0f && p < 1.0f)) return JF_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(mask_bits) & 1u) return JF_ERR_ALIGN;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const float keep_scale = (float)(1.0 / (1.0 - (double)p));
  with_instance<false>(block, N, C, low_dropout(N, C), [&](auto b, auto w, auto r, auto sp) {
    constexpr int B = decltype(b)::value, WAVES = decltype(w)::value, RW = decltype(r)::value;
    hipLaunchKernelGGL((dropout_kernel<B, WAVES, RW, decltype(sp)::value>), (strip_grid<B, WAVES, RW>(N, C)), dim3(64 * WAVES), 0, st, X, SX, mask_bits,
                       keep_scale, (int)N, (int)C, Y, SY);
  });
  return launch_status();
}

extern "C" int32_t jf_add_q(const int8_t* X1, const float* S1, const int8_t* X2, const float* S2, int64_t N, int64_t C,
                            int32_t block, int8_t* Y, float* SY, float* row_mean, float* row_sumsq, void* stream) {
  using namespace jf;
  int32_t rc = check_eltwise(X1, S1, Y, SY, N, C, block);
  if (rc != JF_OK) return rc;
  if (!X2 || !S2) return JF_ERR_NULL;
  if ((row_mean == nullptr) != (row_sumsq == nullptr)) return JF_ERR_NULL;
  if (!aligned16(X2) || !aligned4(S2) || (row_mean && (!aligned4(row_mean) || !aligned4(row_sumsq)))) return JF_ERR_ALIGN;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  with_instance<true>(block, N, C, low_add(block, N, C), [&](auto b, auto w, auto r, auto sp) {
    constexpr int B = decltype(b)::value, WAVES = decltype(w)::value, RW = decltype(r)::value;
    constexpr StorePolicy SP = decltype(sp)::value;
    const auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, (strip_grid<B, WAVES, RW>(N, C)), dim3(64 * WAVES), 0, st, X1, S1, X2, S2, (int)N, (int)C, Y, SY, row_mean, row_sumsq);
    };
    if (row_mean) launch(add_kernel<B, WAVES, RW, true, SP>);
    else launch(add_kernel<B, WAVES, RW, false, SP>);
  });
  return launch_status();
}
