// Fine-grained form of the block-32 product (jf_gemm_kernel.hpp) for outputs of few tiles: 32x32 outputs per workgroup,
// one 16x16 quarter per wave.
//
// The folds of one output element along K are a serial chain, so an output with fewer 32x32 sub-blocks than a few per
// compute unit is bound by the time that a wave alone on its SIMD needs per K step.  A wave that owns 16x16 outputs
// (v_mfma_i32_16x16x32_i8) has 8 vector instructions of fold per K step where the 32x32 sub-block has 32.  512 x 512 at
// K = 2048: 11.8 -> 7.4 us; 1216 x 192 at K = 6912: 28.9 -> 15.5 us.  The price is twice the operand traffic of the 64x64
// tile, so it stops paying once every compute unit has several tiles.
//
// The pipeline: a ring of four stages of 128 bytes of K (eight, which leave room for two workgroups per compute unit instead
// of four, are 9 % slower); the fragments of stage t+1 are read from LDS while stage t is multiplied and folded, so a stage
// costs one barrier and no exposed LDS latency.  Stages, scales and the
// end of the loop are handled as in gemm_tile.
#pragma once
#include "jf_gemm_kernel.hpp"

namespace jf {

template <bool AK, bool BK>
struct FineShape {
  static constexpr int KC = 128, NBUF = 4, NW = 4, TM = 32, TN = 32;
  typedef TileLayout<TM, AK, KC> LA;
  typedef TileLayout<TN, BK, KC> LB;
  static constexpr int A_BYTES = TM * KC, STAGE_BYTES = (TM + TN) * KC;
  static_assert(A_BYTES == 1024 * NW, "one load instruction (64 lanes x 16 bytes) per wave and operand");
  static constexpr int RING_BYTES = NBUF * STAGE_BYTES;
  static constexpr int LDS_BYTES = RING_BYTES + 2 * 2 * 256;   // behind the ring: two segments of 64 scales per operand
};

// 16-wide fragments of 8 bytes per lane: lane l = row l % 16, K bytes 8 * (l / 16) .. + 7 of the K step.
template <bool KMAJOR, int KC>
struct FineFrag {
  typedef TileLayout<32, KMAJOR, KC> L;
  static constexpr int kN = KMAJOR ? KC / 32 : 1;
  int off[kN];
  __device__ __forceinline__ void init(int half, int lane) {
    const int i = lane & 15, g = lane >> 4;
    if (KMAJOR) {
#pragma unroll
      for (int j = 0; j < kN; ++j) off[j] = 16 * L::slot(16 * half + i, 2 * j + (g >> 1)) + 8 * (g & 1);
    } else {
      off[0] = 16 * L::slot(8 * g + (i >> 1), half) + 8 * (i & 1);   // transposing read, see FragAddr
    }
  }
  __device__ __forceinline__ long read(const int8_t* tile, int j) const {
    if (KMAJOR) return *(__attribute__((address_space(3))) long*)(tile + off[j]);
    return __builtin_bit_cast(long, __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(tile + off[0] + j * (32 * L::kCPR * 16))));
  }
};

template <bool AK, bool BK, class LATE>
__device__ __forceinline__ void gemm_fine_tile(GemmArgs g, const int tile_index, const int ntiles, int8_t* const s_ring,
                                               float* const s_amax, LATE&& late) {
  typedef FineShape<AK, BK> S;
  constexpr int B = 32, TM = S::TM, TN = S::TN, KC = S::KC, NBUF = S::NBUF;
  constexpr int SPS = KC / 32;    // K steps (= quantization blocks) per stage
  constexpr int SEG = 64 / SPS;   // stages per segment of 64 scales

  const int tid = threadIdx.x, lane = tid & 63;
  const unsigned wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;   // this wave's quarter

  // tiles to XCDs as in gemm_tile: a contiguous run per XCD, in groups of 8 tile rows
  constexpr int GROUP_M = 8;
  int m0, n0;
  tile_origin<TM, TN, GROUP_M>(tile_index, ntiles, g.M, g.Nn, m0, n0);

  const int nstages = (unsigned)(g.K + KC - 1) / KC, nkb = (unsigned)g.K / B;
  const int last_first = (nstages - 1) * SPS, overlap = nstages > 1 ? nstages * SPS - nkb : 0;   // see gemm_tile
  uint32_t offA = chunk_offset<TM, AK, KC>(wave * 64 + lane, TM, g.K, (uint32_t)g.lda);
  uint32_t offB = chunk_offset<TN, BK, KC>(wave * 64 + lane, TN, g.K, (uint32_t)g.ldb);
  const int8_t* baseA = uniform_pointer(g.A + (AK ? (int64_t)m0 * g.lda : (int64_t)m0));
  const int8_t* baseB = uniform_pointer(g.Bm + (BK ? (int64_t)n0 * g.ldb : (int64_t)n0));
  const int64_t kstrideA = AK ? 1 : g.lda, kstrideB = BK ? 1 : g.ldb;
  int next = 0;   // the stage to request next; past the last one every lane loads one address, so that the counts stay
  auto issue = [&](int slot) __attribute__((always_inline)) {
    if (next >= nstages - 1) {
      if (next == nstages - 1) {
        baseA -= (int64_t)(overlap * B) * kstrideA;
        baseB -= (int64_t)(overlap * B) * kstrideB;
      } else {
        baseA = g.A, offA = 0;
        baseB = g.Bm, offB = 0;
      }
    }
    load_lds_16(baseA, offA, s_ring, slot * S::STAGE_BYTES + 1024 * wave);
    load_lds_16(baseB, offB, s_ring, slot * S::STAGE_BYTES + S::A_BYTES + 1024 * wave);
    baseA += KC * kstrideA;
    baseB += KC * kstrideB;
    ++next;
  };
  // scales of the 64 K blocks of a segment: wave 0 fetches A's, wave 1 B's
  int8_t* const s_scale = s_ring + S::RING_BYTES;
  auto scale_block = [&](int slot) __attribute__((always_inline)) { return slot - (slot >= last_first ? overlap : 0); };
  auto issue_scales = [&](int seg) __attribute__((always_inline)) {
    if (wave < 2) {
      const int kb = min(scale_block(64 * seg + lane), nkb - 1);
      const float* p = wave == 0 ? g.SA + (int64_t)(m0 / B) * g.sa_p + (int64_t)kb * g.sa_k
                                 : g.SB + (int64_t)(n0 / B) * g.sb_p + (int64_t)kb * g.sb_k;
      load_lds_4_vaddr(p, s_scale, ((seg & 1) * 2 + wave) * 256);
    }
  };
  auto read_scales = [&](int seg) __attribute__((always_inline)) -> float {
    typedef __attribute__((address_space(3))) float* lds_f32;
    const int8_t* p = s_scale + (seg & 1) * 512 + 4 * lane;
    const float s = *(lds_f32)(p) * *(lds_f32)(p + 256);
    const int slot = 64 * seg + lane, kb = scale_block(slot);
    return slot < last_first || (kb >= last_first && kb < nkb) ? s : 0.0f;
  };

  FineFrag<AK, KC> fragA;
  FineFrag<BK, KC> fragB;
  fragA.init(wm, lane);
  fragB.init(wn, lane);
  long fa[2][SPS], fb[2][SPS];
  auto read_frags = [&](int slot, int set) __attribute__((always_inline)) {
    const int8_t* ta = s_ring + slot * S::STAGE_BYTES;
#pragma unroll
    for (int j = 0; j < SPS; ++j) {
      fa[set][j] = fragA.read(ta, j);
      fb[set][j] = fragB.read(ta + S::A_BYTES, j);
    }
  };

  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, scales = 0.0f;
  auto compute = [&](int first, int set) __attribute__((always_inline)) {   // first: the stage's first K block in the segment
    v4i v[SPS];
#pragma unroll
    for (int j = 0; j < SPS; ++j) v[j] = __builtin_amdgcn_mfma_i32_16x16x32_i8(fb[set][j], fa[set][j], v4i{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < SPS; ++j)
      fold<0, 4>(acc, v[j], __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, scales), first + j)));
  };
  auto wait_stage = [&](auto stages) __attribute__((always_inline)) {   // as in gemm_tile
    constexpr int N = 2 * decltype(stages)::value;
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
    asm volatile("s_barrier" ::: "memory");
  };

  issue(0);
  late(g);
  issue_scales(0);   // as in gemm_tile
#pragma unroll 1
  for (int t = 1; t < NBUF; ++t) issue(t);
  wait_stage(std::integral_constant<int, NBUF - 1>());
  scales = read_scales(0);
  read_frags(0, 0);
  if (nstages > SEG) issue_scales(1);
  static_assert(NBUF % 2 == 0 && SEG % NBUF == 0, "register sets alternate; segments end with a pass of the loop");
#pragma unroll 1
  for (int t = 0;;) {
    const int first = (t % SEG) * SPS;
    static_for<0, NBUF>([&](auto u) __attribute__((always_inline)) {
      constexpr int i = decltype(u)::value;
      if (t + i < nstages) {
        wait_stage(std::integral_constant<int, NBUF - 2>());
        issue(i);
        read_frags((i + 1) % NBUF, (i + 1) & 1);
        compute(first + i * SPS, i & 1);
      }
    });
    t += NBUF;
    if (t >= nstages) break;
    if (t % SEG == 0) {
      scales = read_scales(t / SEG);
      if (t + SEG < nstages) issue_scales(t / SEG + 1);
    }
  }
  wait_stage(std::integral_constant<int, 0>());   // nothing may land in the ring any more

  // ---- epilogue: max-abs of the block, Eq. 1, codes through LDS so that they are stored as whole rows of the tile.
  // Lane l holds columns 4 * (l / 16) .. + 3 of row l % 16 of the quarter.
  const int row = 16 * wm + (lane & 15), col = 16 * wn + 4 * (lane >> 4);
  if (g.Of) store_part(g.Of + (int64_t)(m0 + row) * g.Nn + n0 + col, make_float4(acc[0], acc[1], acc[2], acc[3]));
  if (!g.Oq) return;
  const float quarter[1] = {fmaxf(fmaxf(fabsf(acc[0]), fabsf(acc[1])), fmaxf(fabsf(acc[2]), fabsf(acc[3])))};
  float amax = wave_max_of<1>(quarter);
  if (lane == 0) s_amax[wave] = amax;
  __syncthreads();
  amax = fmaxf(fmaxf(s_amax[0], s_amax[1]), fmaxf(s_amax[2], s_amax[3]));
  float scale;
  double inv;
  block_scale(amax, scale, inv);
  if (tid == 0) store_out(&g.Os[(int64_t)(m0 / B) * (g.Nn / B) + n0 / B], scale);
  *reinterpret_cast<uint32_t*>(s_ring + row * TN + col) = quantize4(acc[0], acc[1], acc[2], acc[3], inv);
  __syncthreads();
  if (tid < 64) {
    const uint4 v = *reinterpret_cast<const uint4*>(s_ring + 16 * tid);
    store_out(g.Oq + (int64_t)(m0 + tid / 2) * g.Nn + n0 + 16 * (tid & 1), v);
  }
}

// as GemmInstance
template <bool AK, bool BK>
struct FineInstance {
  typedef FineShape<AK, BK> Shape;
  static constexpr int BLOCK = 32;
  static constexpr bool A_KMAJOR = AK, B_KMAJOR = BK;
  static constexpr int WMIN = 4;   // four workgroups per compute unit fit the LDS
  template <class LATE>
  static __device__ __forceinline__ void run(const GemmArgs& g, int tile_index, int ntiles, int8_t* s_ring, float (*s_amax)[8], LATE&& late) {
    gemm_fine_tile<AK, BK>(g, tile_index, ntiles, s_ring, s_amax[0], late);
  }
};

}  // namespace jf
