// Per-block INT8 linear layer (Sec. 5, Alg. 1): forward, dgrad, wgrad and the INT32-partial test hook.
//
// All three products are one kernel in the canonical form  out = A * Bm^T
// (A: M x K, Bm: Nn x K) with two storage modes per operand:
//   K-major  : rows indexed by the output dimension, contraction dimension contiguous
//              (X and W in the forward product, dY in dgrad);
//   M-major  : rows indexed by the contraction dimension (W in dgrad, dY and X in wgrad).
// Tiles are copied global -> LDS unchanged; an M-major tile is transposed
// byte-wise while it is read back with ds_read_b64_tr_b8, so the backward
// products need no separate transpose pass and no re-quantization (square
// blocks: the scale grid is simply indexed with swapped strides).
//
// Per 32-wide K step each wave issues one v_mfma_i32_32x32x32_i8 per 32x32
// output sub-block; at the end of every quantization block along K the INT32
// tile is folded into the FP32 accumulator as fma(sA*sB, (float)v, acc)
// (Sec. 5.3), and after the K loop the accumulator is quantized per block
// (Eq. 1) in registers.  The MFMA operands are swapped (rows of Bm feed the
// "A" port) so that a lane ends up with 4 consecutive output columns of one
// output row per register quad: codes pack into dwords without shuffles.
#pragma once
#include <algorithm>
#include <type_traits>

#include "jf_common.hpp"

namespace jf {

struct GemmArgs {
  const int8_t* A;
  const int8_t* Bm;
  const float* SA;
  const float* SB;
  int M, Nn, K;        // output M x Nn, contraction length K
  int64_t lda, ldb;    // leading dimensions (bytes) of the operands as stored
  int sa_p, sa_k;      // element strides of SA for (output block row, K block)
  int sb_p, sb_k;      // element strides of SB for (output block col, K block)
  int8_t* Oq;          // M x Nn codes (nullable)
  float* Os;           // (M/B) x (Nn/B) scales (nullable with Oq)
  float* Of;           // M x Nn FP32 accumulator (nullable)
  int32_t* dump;       // test hook: INT32 partials of K block dump_kb
  int dump_kb;

  // leading dimensions and scale strides: operands and grids are dense
  __host__ __device__ __forceinline__ void set_strides(int block, bool a_kmajor, bool b_kmajor) {
    lda = a_kmajor ? K : M;
    ldb = b_kmajor ? K : Nn;
    sa_p = a_kmajor ? (unsigned)K / block : 1;
    sa_k = a_kmajor ? 1 : (unsigned)M / block;
    sb_p = b_kmajor ? (unsigned)K / block : 1;
    sb_k = b_kmajor ? 1 : (unsigned)Nn / block;
  }
};

// ---------------------------------------------------------------------------------------------
// LDS staging.  A stage holds KC bytes of K for both operand tiles, 64 (two MFMA K steps) or 128 (see
// GemmShape), so that it always holds whole quantization blocks and block boundaries are known at compile time.  Tiles go global -> LDS with global_load_lds_dwordx4: no VGPR staging, no
// ds_write; the 64 lanes of one such instruction fill 64 consecutive 16-byte LDS slots, so the
// layout cannot be padded.  Bank conflicts are avoided by an XOR swizzle instead: the tile is a
// matrix of 16-byte chunks with CPR chunks per row, and chunk c of row r lives in slot
// r*CPR + (c ^ swz(r)); swz is chosen per operand layout so that the lanes one fragment read serves per
// clock (16 rows for ds_read_b128 of a K-major operand, 8 rows for ds_read_b64_tr_b8 of an M-major one)
// fall into different bank groups.
template <int TILE, bool KMAJOR, int KC>
struct TileLayout {
  static constexpr int kRows = KMAJOR ? TILE : KC;            // LDS rows: output rows, or K rows
  static constexpr int kCPR = (KMAJOR ? KC : TILE) / 16;      // 16-byte chunks per LDS row
  static constexpr int kSlots = kRows * kCPR;
  static_assert(kCPR == 2 || kCPR == 4 || kCPR == 8 || kCPR == 16, "rows of 32, 64, 128 or 256 bytes");
  // K-major tiles are read with ds_read_b128, which serves 16 lanes (16 consecutive rows, one chunk each) per
  // clock from 256 bytes of banks: the 16 rows must land in 16 different 16-byte bank groups.  A row of 128
  // (64) bytes starts at bank group 8*(r%2) (4*(r%4)), so the XOR term has to run through its 8 (4) values
  // over the rows that share that start.  M-major tiles are read with 8-byte transposing reads, 8 rows per
  // 16 lanes: 8 consecutive rows at a fixed chunk cover 8 bank groups.
  static __device__ __forceinline__ int swz(unsigned r) {
    if (KMAJOR) return (r / (16 / kCPR)) % kCPR;
    if (kCPR == 2) return (r / 8) % 2;   // 8 rows cover the banks once, half of them; the next 8 take the other half
    return (r / (kCPR == 4 ? 2 : 1)) % (kCPR == 16 ? 8 : kCPR);
  }
  static __device__ __forceinline__ int slot(int r, int c) { return r * kCPR + (c ^ swz(r)); }
  // LDS bytes when the tile is filled by whole 64-lane load instructions of NW waves (the tail is padding)
  static constexpr int bytes(int nw) { return ((kSlots + 64 * nw - 1) / (64 * nw)) * (64 * nw) * 16; }
};

typedef __attribute__((address_space(3))) v2i* lds_v2i;
typedef __attribute__((address_space(3))) v4i* lds_v4i;

// Per-lane LDS byte offsets of an operand's MFMA fragments inside a stage buffer.  Everything that
// does not depend on the lane is a compile-time immediate added at the read, so the main loop spends
// no vector ALU on addressing.  K-major: the K step j toggles a swizzled chunk bit (one offset per
// j) and the sub-tile adds a constant; M-major: the sub-tile toggles swizzled bits (one offset per
// sub-tile of the wave) and the K step adds a constant.
template <int TILE, bool KMAJOR, int KC, int NSUB>
struct FragAddr {
  typedef TileLayout<TILE, KMAJOR, KC> L;
  static constexpr int kN = KMAJOR ? KC / 32 : NSUB;
  int off[kN];
  __device__ __forceinline__ void init(int sub0, int lane) {
    if (KMAJOR) {
#pragma unroll
      for (int j = 0; j < kN; ++j) off[j] = 16 * L::slot(sub0 * 32 + (lane & 31), 2 * j + (lane >> 5));
    } else {
      // ds_read_b64_tr_b8: within 16 lanes, lane 2r+h points at 8 bytes (columns 8h..8h+7) of row r;
      // lane c receives column c of that 8 x 16 byte matrix.  Two reads give 16 consecutive K.
      const int i = lane & 15, g = lane >> 4;
#pragma unroll
      for (int u = 0; u < kN; ++u)
        off[u] = 16 * L::slot(16 * (g >> 1) + (i >> 1), (sub0 + u) * 2 + (g & 1)) + 8 * (i & 1);
    }
  }
  // fragment of sub-tile u (relative to the wave's first), K step j, from the stage buffer at `tile`
  __device__ __forceinline__ v4i read(const int8_t* tile, int u, int j) const {
    if (KMAJOR) {
      return *(lds_v4i)(tile + off[j] + u * (32 * L::kCPR * 16));
    } else {
      const int8_t* p = tile + off[u] + j * (32 * L::kCPR * 16);
      v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(p));
      v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(p + 8 * L::kCPR * 16));
      v4i r = {lo[0], lo[1], hi[0], hi[1]};
      return r;
    }
  }
};

// Byte offset, from the tile's origin at the stage's start, of the chunk that belongs in LDS slot `slot_idx`.  Rows or
// columns outside the matrix (outer_left: from the origin to its edge) and K beyond klim are clamped to valid addresses:
// what they deliver only reaches outputs that are never stored, or K blocks of scale 0, so no zero fill is needed.
template <int TILE, bool KMAJOR, int KC>
__device__ __forceinline__ uint32_t chunk_offset(unsigned slot_idx, unsigned outer_left, unsigned klim, uint32_t ld) {
  typedef TileLayout<TILE, KMAJOR, KC> L;
  const unsigned r = min(slot_idx / L::kCPR, L::kRows - 1u);  // slots past the tile are padding: any valid source will do
  const unsigned c = (slot_idx % L::kCPR) ^ L::swz(r);
  return KMAJOR ? min(r, outer_left - 1) * ld + min(16 * c, klim - 16) : min(r, klim - 1) * ld + min(16 * c, outer_left - 16);
}

// The lane's number, computed where it is needed, so that neither it nor what follows from it takes a register through the K loop (where
// one too many goes to scratch memory, whose loads wait for the stages in flight: weight gradient 735 -> 796 us).
__device__ __forceinline__ int lane_again() {
  int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  asm volatile("" : "+v"(lane));
  __builtin_assume(lane >= 0 && lane < 64);
  return lane;
}

// f(integral_constant<int, I>) for I = BEGIN .. END-1, unrolled at compile time
template <int BEGIN, int END, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (BEGIN < END) {
    f(std::integral_constant<int, BEGIN>());
    static_for<BEGIN + 1, END>(f);
  }
}

// acc += t * (float)v for one 32x32 sub-block (Sec. 5.3), t in a scalar register: 16 int->float conversions and 16 FMAs
// per lane.  The fused multiply-add is written as v_fmac_f32 so that it updates the accumulator register in place;
// left to itself the register allocator ping-pongs the 64 accumulators between two register sets.
template <int R0, int R1, class V, int N>
__device__ __forceinline__ void fold(float (&acc)[N], const V& v, float t) {
#pragma unroll
  for (int r = R0; r < R1; ++r) {
    const float c = (float)v[r];
    asm("v_fmac_f32 %0, %1, %2" : "+v"(acc[r]) : "s"(t), "v"(c));
  }
}
// The same in two halves, for loops that keep them apart.
__device__ __forceinline__ void fold_convert(float (&c)[16], const v16i& v) {
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] = (float)v[r];
}
__device__ __forceinline__ void fold_add(float (&acc)[16], const float (&c)[16], float t) {
#pragma unroll
  for (int r = 0; r < 16; ++r) asm("v_fmac_f32 %0, %1, %2" : "+v"(acc[r]) : "s"(t), "v"(c[r]));
}

// First row and column of the tile that a workgroup takes.  Workgroups are dealt round-robin to the 8 XCDs (each with its own
// L2).  Renumber them so that every XCD works on one contiguous run of tiles, and order the tiles in groups of GROUP_M tile rows,
// column by column inside a group: the workgroups that are resident on an XCD at the same time then form a compact patch
// (GROUP_M tile rows x a few tile columns) that re-reads few distinct operand tiles from that XCD's L2.
// All of it stands in front of a tile's first load, one instruction after the other: unsigned, and one division in all groups but
// the last (with the lane offsets of the loads unsigned too, 50 of the 310 instructions in front of the first stage: 1024^3
// 6.8 -> 6.65 us, 1056 x 800 -> 2080 8.7 -> 8.5).
template <int TM, int TN, int GROUP_M>
__device__ __forceinline__ void tile_origin(unsigned index, unsigned ntiles, int M, int Nn, int& m0, int& n0) {
  const unsigned tiles_n = (unsigned)(Nn + TN - 1) / TN, tiles_m = (unsigned)(M + TM - 1) / TM;
  const unsigned xcd = index & 7, tile = xcd * (ntiles >> 3) + min(xcd, ntiles & 7) + (index >> 3);
  const unsigned group = tile / (GROUP_M * tiles_n), in_group = tile - group * GROUP_M * tiles_n;
  const unsigned first_m = group * GROUP_M, group_rows = tiles_m - first_m;
  unsigned row = in_group % GROUP_M, col = in_group / GROUP_M;
  if (group_rows < GROUP_M) row = in_group % group_rows, col = in_group / group_rows;   // the last group
  m0 = (int)((first_m + row) * TM);
  n0 = (int)(col * TN);
}

// Compile-time shape of one kernel instance: tile, stage and LDS ring.
template <int B, int WM, int WN, int WGM, int WGN, bool AK, bool BK>
struct GemmShape {
  static constexpr int NW = WGM * WGN;
  static constexpr int TM = 32 * WM * WGM, TN = 32 * WN * WGN;
  // K bytes per stage: 128 when a stage has to hold a whole B = 128 block, and for the waves of one sub-block, which
  // spend the most instructions per MFMA on the stage itself (at B = 64 a stage must also hold an even number of sub-block
  // x K-block units); 64 otherwise, which lets three workgroups with a ring of three stages share the LDS of a compute unit.
  static constexpr int KC = (B == 128 || WM * WN == 1) ? 128 : 64;
  typedef TileLayout<TM, AK, KC> LA;
  typedef TileLayout<TN, BK, KC> LB;
  static constexpr int A_BYTES = LA::bytes(NW), B_BYTES = LB::bytes(NW);
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  // Stages in the LDS ring: one being read, the rest in flight.  Two for the waves of one sub-block at B = 32: with four
  // workgroups per compute unit a stage lasts long enough (2048^3, forward / dgrad / wgrad: 22.0 / 20.9 / 22.7 us
  // against 23.5 / 22.2 / 22.7 with three stages of 64 bytes; 4096 x 768 -> 3072 27.2 / 23.3 / 29.8 against 29.4 / 25.8 / 30.0;
  // three stages of 128 bytes leave room for three workgroups and are slower).  Tiles that leave a compute unit to a single
  // workgroup (more than four waves, B > 32) take four if that fits the LDS, the others three.
  static constexpr int NBUF = (B == 32 && WM * WN == 1) ? 2 : (B > 32 && NW > 4 && 4 * STAGE_BYTES <= 156 * 1024) ? 4 : 3;
  static_assert(NBUF * STAGE_BYTES <= 156 * 1024, "the ring must fit the LDS of a compute unit");
  static constexpr int RING_BYTES = NBUF * STAGE_BYTES;
  // Block scales: two segments of 64 K blocks for every block row and block column of the tile, behind the ring.
  static constexpr int SCALE_ROWS_A = (TM + B - 1) / B, SCALE_ROWS = SCALE_ROWS_A + (TN + B - 1) / B;
  static constexpr int LDS_BYTES = RING_BYTES + 2 * SCALE_ROWS * 256;
};

// How a wave reads its fragments (see the pipeline in gemm_tile): per K step where a stage holds several quantization blocks
// and the wave several sub-blocks; else per stage, in one register set where two do not fit (2x2 sub-blocks at three waves
// per SIMD).
template <int B, int WM, int WN>
struct GemmPipeline {
  static constexpr bool STEPWISE = B == 32, ONE_SET = B == 64 && WM * WN > 1;
};

// One output tile: K loop and epilogue.  `tile_index` of `ntiles` is this workgroup's position in the launch (or in
// its part of a launch that holds two products); s_ring is the workgroup's LDS ring of NBUF stages with the scales behind
// it, s_amax its max-abs exchange area, both owned by the calling kernel.  late(g) completes the arguments by those that are not
// needed for the first stage's loads, behind which it is called.
template <int B, int WM, int WN, int WGM, int WGN, bool AK, bool BK, bool DUMP, class LATE>
__device__ __forceinline__ void gemm_tile(GemmArgs g, const int tile_index, const int ntiles, int8_t* const s_ring,
                                          float (*const s_amax)[8], LATE&& late) {
  typedef GemmShape<B, WM, WN, WGM, WGN, AK, BK> Shape;
  constexpr int NW = Shape::NW;
  constexpr int TM = Shape::TM, TN = Shape::TN;
  constexpr int KPB = B / 32;  // MFMA K steps per quantization block
  constexpr int KC = Shape::KC;
  constexpr int SPS = KC / 32;  // MFMA K steps per stage
  constexpr int NTILE = WM * WN;
  typedef typename Shape::LA LA;
  typedef typename Shape::LB LB;
  constexpr int A_BYTES = Shape::A_BYTES, B_BYTES = Shape::B_BYTES;
  constexpr int CA = A_BYTES / (1024 * NW), CB = B_BYTES / (1024 * NW);  // load instructions per wave and stage
  static_assert(B == 32 || (TM % B == 0 && TN % B == 0), "tile must hold whole quantization blocks");
  constexpr int STAGE_BYTES = Shape::STAGE_BYTES;
  constexpr int NBUF = Shape::NBUF;
  static_assert(TM / 32 <= 8 && TN / 32 <= 8, "max-abs exchange area");
  int8_t* const s_tile0 = s_ring;
  int8_t* const s_tile1 = s_ring + STAGE_BYTES;
  int8_t* const s_tile2 = s_ring + 2 * STAGE_BYTES;
  int8_t* const s_tile3 = s_ring + (NBUF > 3 ? 3 : 2) * STAGE_BYTES;
  auto tile_buf = [&](int buf) -> int8_t* {
    return buf == 0 ? s_tile0 : (buf == 1 ? s_tile1 : (buf == 2 ? s_tile2 : s_tile3));
  };

  const int tid = threadIdx.x, lane = tid & 63;
  const unsigned wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;  // first 32-granule of this wave inside the tile

  // 256x128 at B = 32, 128 registers for 64 accumulators and two INT32 tiles: five others went to scratch memory, the lane's number among them
  constexpr bool LANE_AGAIN = B == 32 && NW == 8 && NTILE == 4;
  constexpr int GROUP_M = TM >= 256 ? 4 : 8;
  int m0, n0;
  tile_origin<TM, TN, GROUP_M>(tile_index, ntiles, g.M, g.Nn, m0, n0);

  const int nstages = (unsigned)(g.K + KC - 1) / KC, nkb = (unsigned)g.K / B;
  constexpr int NKB = SPS / KPB;  // quantization blocks along K per stage
  // Stages are whole: when K is not a multiple of KC the last one starts earlier, `overlap` blocks back, at K - KC, and
  // the blocks it shares with the one before it carry scale 0.  (A K shorter than one stage is clamped in the lane
  // offsets instead; what the clamped lanes deliver belongs to blocks beyond K, which carry scale 0 as well.)
  const int last_first = (nstages - 1) * NKB, overlap = nstages > 1 ? nstages * NKB - nkb : 0;

  // A load's address is a workgroup-uniform base (the tile's origin, advanced by KC (K-major) or KC*ld (M-major)
  // per stage with scalar instructions) plus a loop-invariant per-lane byte offset.  The offset fits 32 bits: a
  // tile spans at most 256 rows (or 128 K rows) of at most 2^24 + 32 bytes.  The load takes them as scalar base
  // + vector offset, so the K loop spends no vector ALU on addresses.
  uint32_t offA[CA], offB[CB];
  const int64_t originA = AK ? (int64_t)m0 * g.lda : (int64_t)m0, originB = BK ? (int64_t)n0 * g.ldb : (int64_t)n0;
#pragma unroll
  for (int i = 0; i < CA; ++i) offA[i] = chunk_offset<TM, AK, KC>((i * NW + wave) * 64 + lane, g.M - m0, g.K, (uint32_t)g.lda);
#pragma unroll
  for (int i = 0; i < CB; ++i) offB[i] = chunk_offset<TN, BK, KC>((i * NW + wave) * 64 + lane, g.Nn - n0, g.K, (uint32_t)g.ldb);
  const int8_t* baseA = uniform_pointer(g.A + originA);
  const int8_t* baseB = uniform_pointer(g.Bm + originB);
  const int64_t kstrideA = AK ? 1 : g.lda, kstrideB = BK ? 1 : g.ldb;
  // Issue the direct-to-LDS loads of the next stage into ring slot `slot`, one at a time.  There is no separate code for the end of the
  // loop: past the last stage every lane loads the same valid address, so that the counts of outstanding loads never
  // change.  (The straight-line tails this replaces made the kernels 3-4 times as long, and code that runs once is
  // fetched once: 64 KB of it cost a product of 12 stages 2 us.)
  constexpr int LOADS = CA + CB;   // vector-memory instructions per wave and stage
  int next = 0;
  auto issue_load = [&](int slot, int n) __attribute__((always_inline)) {   // load n of stage `next`
    if (n == 0 && next >= nstages - 1) {
      if (next == nstages - 1) {
        baseA -= (int64_t)(overlap * B) * kstrideA;
        baseB -= (int64_t)(overlap * B) * kstrideB;
      } else {
        baseA = g.A;
        baseB = g.Bm;
#pragma unroll
        for (int i = 0; i < CA; ++i) offA[i] = 0;
#pragma unroll
        for (int i = 0; i < CB; ++i) offB[i] = 0;
      }
    }
    const int byte = slot * STAGE_BYTES + 1024 * wave;
    if (n < CA) load_lds_16(baseA, offA[n], s_ring, byte + 1024 * n * NW);
    else load_lds_16(baseB, offB[n - CA], s_ring, byte + A_BYTES + 1024 * (n - CA) * NW);
    if (n + 1 == LOADS) {
      baseA += KC * kstrideA;
      baseB += KC * kstrideB;
      ++next;
    }
  };

  FragAddr<TM, AK, KC, WM> addrA;
  FragAddr<TN, BK, KC, WN> addrB;
  addrA.init(wm0, lane);
  addrB.init(wn0, lane);

  float acc[WM][WN][16];
  const v16i zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

  auto dump_tile = [&](const v16i& v, int a, int b) __attribute__((always_inline)) {
    const int m = m0 + 32 * (wm0 + a) + (lane & 31);
    const int nb = n0 + 32 * (wn0 + b) + 4 * (lane >> 5);
    if (m < g.M && nb < g.Nn) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        v4i o = {v[4 * q4], v[4 * q4 + 1], v[4 * q4 + 2], v[4 * q4 + 3]};
        *reinterpret_cast<v4i*>(g.dump + (int64_t)m * g.Nn + nb + 8 * q4) = o;
      }
    }
  };

  // Stage loop over the ring of NBUF LDS buffers: while stage t is computed, stages t+1 .. t+NBUF-1 are in flight,
  // which covers the L2 latency even when a stage is only two K steps long.  The loop is unrolled NBUF times so that every
  // LDS address is a compile-time immediate and the accumulators stay in the same registers.
  static_assert(LOADS * (NBUF - 1) <= 63, "vmcnt immediate");
  // Wait for this wave's own loads of all but the youngest `stages` stages and for its LDS reads, then meet the other
  // waves.  A bare s_barrier is used instead of __syncthreads(): the fence of the latter makes the compiler drain
  // every outstanding load (vmcnt(0)), including the stages that are meant to stay in flight.  Ordering is kept
  // by hand: the asm is a compiler barrier for memory accesses, each wave has consumed all its LDS reads of the
  // finished stage before it arrives, and direct-to-LDS loads are counted by vmcnt.  The wait itself is the
  // s_waitcnt builtin, which the compiler's own counter tracking understands.
  // (The test hook's stores are counted by vmcnt too, and not in order with the loads, so it always drains.  A load of
  // scales among the outstanding ones makes the wait stricter.)
  auto wait_stage = [&](auto stages) __attribute__((always_inline)) {
    // s_waitcnt immediate: vmcnt in bits 3:0 and 15:14, expcnt (6:4) left at "no wait", lgkmcnt (11:8) 0
    constexpr int N = DUMP ? 0 : LOADS * decltype(stages)::value;
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
    asm volatile("s_barrier" ::: "memory");
  };

  // ---- Block scales.  Lane k of a register per sub-block holds sA * sB of K block k of the current segment; one
  // v_readlane per K block and sub-block turns it into the scalar operand of the folds (33 vector instructions per
  // sub-block and K block; from scalar loads it took a v_mov and a v_mul, 34, and twelve scalar instructions per stage).
  // A segment is a whole number of passes of the stage loop; the waves fetch its scales into LDS one segment ahead.
  constexpr int UNROLL = GemmPipeline<B, WM, WN>::STEPWISE || GemmPipeline<B, WM, WN>::ONE_SET || NBUF % 2 == 0 ? NBUF : 2 * NBUF;   // stages per pass
  constexpr int PASS = UNROLL * NKB, SEG = (64 / PASS) * PASS;
  int8_t* const s_scale = s_ring + Shape::RING_BYTES;
  auto scale_block = [&](int slot) __attribute__((always_inline)) {   // K block of block slot `slot` (stages are whole)
    return slot - (slot >= last_first ? overlap : 0);
  };
  auto issue_scales = [&](int seg) __attribute__((always_inline)) {
    if (DUMP) return;
    const int lane = LANE_AGAIN ? lane_again() : tid & 63, kb = min(scale_block(seg * SEG + lane), nkb - 1);
#pragma unroll
    for (int r0 = 0; r0 < Shape::SCALE_ROWS; r0 += NW) {
      const int r = r0 + (int)wave;
      if (r < Shape::SCALE_ROWS) {
        const int rb = r - Shape::SCALE_ROWS_A;
        const float* p = rb < 0 ? g.SA + (int64_t)((unsigned)min(m0 + B * r, g.M - B) / B) * g.sa_p + (int64_t)kb * g.sa_k
                                : g.SB + (int64_t)((unsigned)min(n0 + B * rb, g.Nn - B) / B) * g.sb_p + (int64_t)kb * g.sb_k;
        load_lds_4_vaddr(p, s_scale, ((seg & 1) * Shape::SCALE_ROWS + r) * 256);
      }
    }
  };
  float scales[WM][WN];
  auto read_scales = [&](int seg) __attribute__((always_inline)) {
    if (DUMP) return;
    typedef __attribute__((address_space(3))) float* lds_f32;
    const int lane = LANE_AGAIN ? lane_again() : tid & 63;
    const int8_t* p = s_scale + (seg & 1) * Shape::SCALE_ROWS * 256 + 4 * lane;
    const int slot = seg * SEG + lane, kb = scale_block(slot);
    const bool counts = slot < last_first || (kb >= last_first && kb < nkb);
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
      for (int b = 0; b < WN; ++b) {
        const float sa = *(lds_f32)(p + 256 * (32 * (wm0 + a) / B));
        const float sb = *(lds_f32)(p + 256 * (Shape::SCALE_ROWS_A + 32 * (wn0 + b) / B));
        scales[a][b] = counts ? sa * sb : 0.0f;
      }
  };

  // ---- One software pipeline per wave that runs across the stage barriers.  The unit is the product of one
  // 32x32 sub-block with one quantization block along K: a chain of KPB MFMAs into one INT32 tile, then the
  // fold of that tile into the FP32 accumulator (32 conversions/FMAs; at B = 32 the kernel is bound by them).
  // Two INT32 tiles rotate: the chain of the next unit is issued before the fold of the current one.
  // Fragments are read from LDS ahead of the chain that takes them and spread over the folds, one or two reads per unit:
  // read all at once after the barrier they hold up the vector ALU, which they share register ports with.
  //   STEPWISE (B = 32): the fragments of one K step are read while the units of the K step before are folded (two steps
  //     before, where a step is a single unit); two register sets used by turns.  The barrier stands before the last step(s).
  //   ONE_SET (2x2 sub-blocks at B = 64, where two sets do not fit three waves per SIMD): those of the next stage into
  //     the registers that come out of use, beside the last two units.  The barrier stands before them.
  //   otherwise: those of one stage while the stage before is folded; two sets, one per stage.  The barrier comes first.
  static_assert(SPS % KPB == 0 && (NKB * NTILE) % 2 == 0, "a stage leaves the tile rotation where it found it");
  constexpr int NT = NKB * NTILE;   // units per stage
  constexpr bool STEPWISE = GemmPipeline<B, WM, WN>::STEPWISE, ONE_SET = GemmPipeline<B, WM, WN>::ONE_SET;
  static_assert(!STEPWISE || (KPB == 1 && SPS % 2 == 0), "the register sets alternate");
  static_assert(!ONE_SET || (WM == 2 && WN == 2 && NT == 4), "the order in which fragments come out of use");
  // Two waves of a workgroup on every SIMD: priorities fall from one meeting of the waves to the next instead of over the whole loop,
  // so that the two arrive together (256x128 tiles: 8192^3 at B = 32 990 / 986 / 959 -> 982 / 975 / 947 us, 4096 x 4096 -> 2048 at B = 128
  // forward 41.6 -> 40.1; eight waves of one sub-block, six to a SIMD, gain 1 % alone and lose 1.4 as a pair).
  constexpr bool BY_STAGE = NW == 8 && NTILE > 1;
  constexpr int SETS = STEPWISE || !ONE_SET ? 2 : 1, STEPS = STEPWISE ? 1 : SPS;   // register sets, K steps in each
  constexpr int AHEAD = NTILE == 1 ? 2 : 1;   // STEPWISE: K steps between a read and the step beside which it stands
  v16i vi[2];
  v4i fa[SETS][STEPS][WM], fb[SETS][STEPS][WN];
  constexpr int READS = WM + WN;
  // read number n of K step j of the stage in ring slot `slot`
  auto read_frag = [&](int slot, int set, int j, int n) __attribute__((always_inline)) {
    const int8_t* ta = tile_buf(slot);
    if (n < WM) fa[set][STEPWISE ? 0 : j][n] = addrA.read(ta, n, j);
    else fb[set][STEPWISE ? 0 : j][n - WM] = addrB.read(ta + A_BYTES, n - WM, j);
  };
  // registers [16*part/KPB, 16*(part+1)/KPB) of unit i's fold (the test hook stores the whole tile at part 0)
  auto fold_or_dump = [&](int t, int i, const v16i& v, float scale, auto part_tag) __attribute__((always_inline)) {
    constexpr int part = decltype(part_tag)::value;
    const int a = (i % NTILE) / WN, b = (i % NTILE) % WN;
    if (DUMP) {
      if (part == 0 && scale_block(t * NKB + i / NTILE) == g.dump_kb) dump_tile(v, a, b);
    } else {
      fold<16 * part / KPB, 16 * (part + 1) / KPB>(acc[a][b], v, scale);
    }
  };
  // MFMA number js of the chain of unit i of a stage (quantization block i / NTILE, sub-block i % NTILE) into dst
  auto chain_step = [&](int set, int i, int js, v16i& dst) __attribute__((always_inline)) {
    const int kb = i / NTILE, a = (i % NTILE) / WN, b = (i % NTILE) % WN;
    const int st = STEPWISE ? kb % 2 : set, j = STEPWISE ? 0 : kb * KPB + js;
    dst = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[st][j][b], fa[st][j][a], js == 0 ? zero16 : dst, 0, 0, 0);
  };
  int first = 0;        // block slot of the pass's first block inside the segment
  float scale = 0.0f;   // of the unit to be folded next; read one unit ahead
  auto scale_of = [&](int slot, int i) __attribute__((always_inline)) {   // unit i of the stage that starts at block slot `slot` of the segment
    if (DUMP) return 0.0f;
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, scales[(i % NTILE) / WN][(i % NTILE) % WN]), slot + i / NTILE));
  };
  // Stage t out of ring slot u % NBUF, u its place in the pass; on entry the fragments of its first K step (STEPWISE) or all
  // of them are in registers and the chain of its first unit is in flight in vi[0], on return the same for the next stage.
  // Beside the fold of each unit: the chain of the next unit, each MFMA of it (32 cycles of the matrix pipe) followed by
  // 32/KPB vector instructions (4 cycles each), so that a single wave keeps both pipes busy.
  auto run_stage = [&](int t, auto u_tag) __attribute__((always_inline)) {
    constexpr int u = decltype(u_tag)::value, slot = u % NBUF, nslot = (u + 1) % NBUF;
    constexpr int set = ONE_SET ? 0 : u & 1, nset = ONE_SET ? 0 : set ^ 1;
    constexpr int SYNC = STEPWISE ? (SPS - AHEAD) * NTILE : ONE_SET ? NT - 2 : 0;   // the unit before which the waves meet
    constexpr bool SPREAD_LOADS = B == 128;
    static_for<0, NT>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value, kb = i / NTILE, q = i % NTILE;
      v16i &cur = vi[i & 1], &nxt = vi[(i & 1) ^ 1];
      if constexpr (BY_STAGE) {
        constexpr int done = (i - SYNC + NT) % NT;   // units since the last meeting
        if constexpr (done == 0 || 4 * done / NT != 4 * (done - 1) / NT) __builtin_amdgcn_s_setprio(3 - 4 * done / NT);
      }
      if constexpr (i == SYNC) wait_stage(std::integral_constant<int, NBUF - 2>());
      // The loads of the stage NBUF ahead, into the slot that this one has left: all at once, or, from the eight waves of
      // a compute unit's only workgroup, one after another over the units -- requested together they wait for each other
      // there, and the MFMAs behind them with them (8192 x 4096 -> 8192 at B = 128 320 -> 312 us; the other shapes, whose
      // workgroups are out of step, lose 1-5 % by it).
      auto loads = [&](auto js_tag) __attribute__((always_inline)) {
        constexpr int p0 = SYNC * KPB, P = SPREAD_LOADS ? NT * KPB - p0 : 1, at = i * KPB + decltype(js_tag)::value - p0;
        static_for<0, LOADS>([&](auto n) __attribute__((always_inline)) {
          if constexpr (decltype(n)::value * P / LOADS == at) issue_load(slot, decltype(n)::value);
        });
      };
      if constexpr (!SPREAD_LOADS) loads(std::integral_constant<int, 0>());
      const float s = scale;
      scale = scale_of(first + u * NKB, i + 1);
      static_for<0, KPB>([&](auto js_tag) __attribute__((always_inline)) {
        constexpr int js = decltype(js_tag)::value;
        if constexpr (i + 1 < NT) chain_step(set, i + 1, js, nxt);
        else chain_step(nset, 0, js, nxt);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (STEPWISE && AHEAD == 2) {   // the K step after next, into the registers of this one
          static_for<0, READS>([&](auto n_tag) __attribute__((always_inline)) {
            read_frag(kb + 2 < SPS ? slot : nslot, kb % 2, (kb + 2) % SPS, decltype(n_tag)::value);
          });
        } else if constexpr (STEPWISE) {   // the next K step's reads: all but the last unit of this one share them
          constexpr int U = NTILE - 1;
          static_for<0, READS>([&](auto n_tag) __attribute__((always_inline)) {
            constexpr int n = decltype(n_tag)::value;
            if constexpr (n * U / READS == q) read_frag(kb + 1 < SPS ? slot : nslot, (kb + 1) % 2, (kb + 1) % SPS, n);
          });
        } else if constexpr (ONE_SET) {
          // the next stage's, as this one's come out of use: those of sub-block 0 beside the last unit but one, the
          // rest, which the chain issued in that unit has read, beside the last
          static_for<0, SPS>([&](auto j_tag) __attribute__((always_inline)) {
            constexpr int j = decltype(j_tag)::value;
            if constexpr (j % KPB == js && i == NT - 2) read_frag(nslot, 0, j, 0), read_frag(nslot, 0, j, WM);
            if constexpr (j % KPB == js && i == NT - 1) read_frag(nslot, 0, j, 1), read_frag(nslot, 0, j, WM + 1);
          });
        } else {   // the next stage's reads, over all but the last unit and the MFMAs of their chains
          constexpr int P = (NT - 1) * KPB, R = SPS * READS;
          static_for<0, R>([&](auto n_tag) __attribute__((always_inline)) {
            constexpr int n = decltype(n_tag)::value;
            if constexpr (n * P / R == i * KPB + js) read_frag(nslot, nset, n / READS, n % READS);
          });
        }
        if constexpr (SPREAD_LOADS) loads(js_tag);
        fold_or_dump(t, i, cur, s, js_tag);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };

  static_assert(NBUF >= 2, "a stage in flight beside the one in use");
  const auto issue_stage = [&](int t) __attribute__((always_inline)) {
    static_for<0, LOADS>([&](auto n) __attribute__((always_inline)) { issue_load(t, decltype(n)::value); });
  };
  issue_stage(0);
  late(g);
  issue_scales(0);   // the wait for the first stage takes them in
#pragma unroll 1
  for (int t = 1; t < NBUF; ++t) issue_stage(t);
  // while the first stage is on its way (the compiler would do it behind the wait, 64 instructions of every wave of a SIMD)
#pragma unroll
  for (int a = 0; a < WM; ++a)
#pragma unroll
    for (int b = 0; b < WN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) asm volatile("v_mov_b32 %0, 0" : "=v"(acc[a][b][r]));
  wait_stage(std::integral_constant<int, NBUF - 1>());
  static_for<0, (STEPWISE ? AHEAD : STEPS) * READS>([&](auto n) __attribute__((always_inline)) {
    constexpr int j = decltype(n)::value / READS;
    read_frag(0, STEPWISE ? j : 0, j, decltype(n)::value % READS);
  });
  read_scales(0);
  if (nkb > SEG) issue_scales(1);
  static_for<0, KPB>([&](auto js) __attribute__((always_inline)) { chain_step(0, 0, decltype(js)::value, vi[0]); });
  scale = scale_of(0, 0);
#pragma unroll 1
  for (int t = 0, seg = 0;;) {
    // The instruction arbiter favours the oldest wave of a SIMD, so co-resident waves would finish one after
    // the other and leave the SIMD to a single wave at the end.  Each wave therefore lowers its own priority
    // as it advances: whoever is ahead yields, and the waves of a SIMD reach the end together.
    if (BY_STAGE) {
    } else if (4 * t < nstages) __builtin_amdgcn_s_setprio(3);
    else if (2 * t < nstages) __builtin_amdgcn_s_setprio(2);
    else if (4 * t < 3 * nstages) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
    static_for<0, UNROLL>([&](auto u) __attribute__((always_inline)) {
      if (t + decltype(u)::value < nstages) run_stage(t + decltype(u)::value, u);
    });
    t += UNROLL;
    if (t >= nstages) break;
    first += PASS;
    if (first == SEG) {
      first = 0;
      read_scales(++seg);
      if ((seg + 1) * SEG < nstages * NKB) issue_scales(seg + 1);
      scale = scale_of(0, 0);
    }
  }
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_s_waitcnt(7 << 4 | 15 << 8);   // vmcnt 0: nothing may land in the ring any more
  if (DUMP) return;

  // ---- epilogue: optional FP32 store, per-block max-abs, Eq. 1, packed INT8 store.  Vector-ALU work like the loop, and the last
  // workgroup's has nothing beside it: the maxima of the wave's blocks are reduced together and Eq. 1's scale is computed once for all
  // of them (four blocks: 600 -> 470 instructions, 4096 x 768 -> 3072 23.85 -> 23.2 us, 8192 x 1280 -> 5120 112 -> 110).
  const int lane_out = LANE_AGAIN ? lane_again() : lane, tid_out = LANE_AGAIN ? (int)(64 * wave) + lane_out : tid;
  // Pieces of quantization blocks that this wave holds: at B = 32 its sub-blocks, else one, whole or shared with other waves.
  constexpr int PM = WM * 32 < B ? WM : B / 32, PN = WN * 32 < B ? WN : B / 32, PIECES_N = WN / PN, PIECES = WM / PM * PIECES_N;
  float piece[PIECES];
#pragma unroll
  for (int k = 0; k < PIECES; ++k) {
    piece[k] = 0.0f;
#pragma unroll
    for (int a = 0; a < PM; ++a)
#pragma unroll
      for (int b = 0; b < PN; ++b) piece[k] = amax16(piece[k], acc[k / PIECES_N * PM + a][k % PIECES_N * PN + b]);
  }
  float amax = wave_max_of<PIECES>(piece);   // of the lane's piece
  if constexpr (PM * 32 < B || PN * 32 < B) {
    static_assert(PIECES == 1, "the waves of a block exchange one value each");
    if (lane_out == 0) s_amax[wm0][wn0] = amax;
    __syncthreads();
    constexpr int G = B / 32;
    const int ga = wm0 / G * G, gb = wn0 / G * G;
#pragma unroll
    for (int x = 0; x < G; x += WM)
#pragma unroll
      for (int y = 0; y < G; y += WN) amax = fmaxf(amax, s_amax[ga + x][gb + y]);
  }
  float scale_out = 0.0f;
  double inv_out = 0.0;
  if (g.Oq) {
    block_scale(amax, scale_out, inv_out);
    const int k = lane_value<PIECES>(lane_out), row = m0 + 32 * (wm0 + k / PIECES_N * PM), col = n0 + 32 * (wn0 + k % PIECES_N * PN);
    if (lane_out == value_lane<PIECES>(k) && row < g.M && col < g.Nn && row % B == 0 && col % B == 0)
      store_out(&g.Os[(int64_t)(row / B) * (g.Nn / B) + col / B], scale_out);
  }
  if constexpr (!AK && !BK) if (g.Of && !g.Oq) {
    // FP32 results alone, the gradient of a master weight (no other product is asked for them, and even unused the code costs 1056 x 800 -> 2080
    // forward 8.3 -> 8.55 us): a lane has 16 bytes of a row at a time, the other half wave the next 16, so each wave
    // turns its sub-blocks in 4 KB of the ring and stores whole lines, eight rows an instruction (chunks swizzled by the row: rows of 128
    // bytes start at the same bank).  2048^3 22.7 -> 20.5 us, 448 x 4448 -> 8384 59.7 -> 54.3, 512 x 1024 -> 1024
    // 5.06 -> 4.74.
    static_assert(Shape::RING_BYTES >= 4096 * NW, "4 KB of the ring for each wave");
    __syncthreads();   // (the ring, as below)
    int8_t* const turn = s_ring + 4096 * wave;
    const int r = lane_out & 31;
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
      for (int b = 0; b < WN; ++b) {
        const int mrow0 = m0 + 32 * (wm0 + a), ncol0 = n0 + 32 * (wn0 + b);
        if (mrow0 >= g.M || ncol0 >= g.Nn) continue;   // the same for the whole wave
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *reinterpret_cast<float4*>(turn + 128 * r + 16 * ((2 * q4 + (lane_out >> 5)) ^ (r & 7))) =
              make_float4(acc[a][b][4 * q4], acc[a][b][4 * q4 + 1], acc[a][b][4 * q4 + 2], acc[a][b][4 * q4 + 3]);
        // a wave's own LDS accesses are served in order; the fences keep the compiler to it
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        float* const out = g.Of + (int64_t)mrow0 * g.Nn + ncol0 + 4 * (lane_out & 7);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const int row = 8 * p + (lane_out >> 3);
          store_out(out + (int64_t)row * g.Nn, *reinterpret_cast<const v4f*>(turn + 128 * row + 16 * ((lane_out & 7) ^ (row & 7))));
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    return;
  }
  // The code tile is staged in the operand ring: in one slot, or split by rows over two slots when a slot is
  // smaller than the tile.  The last stage of the K loop ends without a barrier, so a wave may still be reading its
  // fragments of that stage out of the ring while a faster one is already here: meet once before the ring is
  // overwritten (where waves share a block, the barrier of the max-abs exchange above has done that).
  if (PM * 32 >= B && PN * 32 >= B && g.Oq != nullptr) __syncthreads();
  constexpr int CODE_ROWS_PER_SLOT = TM * TN <= STAGE_BYTES ? TM : TM / 2;
  static_assert(CODE_ROWS_PER_SLOT * TN <= STAGE_BYTES, "half the code tile fits a ring slot");
  auto code_row = [&](int row) __attribute__((always_inline)) -> int8_t* {
    return (row < CODE_ROWS_PER_SLOT ? s_tile0 : s_tile1) + (row % CODE_ROWS_PER_SLOT) * TN;
  };
#pragma unroll
  for (int a = 0; a < WM; ++a)
#pragma unroll
    for (int b = 0; b < WN; ++b) {
      const int mrow0 = m0 + 32 * (wm0 + a), ncol0 = n0 + 32 * (wn0 + b);
      if (mrow0 >= g.M || ncol0 >= g.Nn) continue;  // wave-uniform: the whole sub-block is outside
      const int m = mrow0 + (lane_out & 31);
      const int nb = ncol0 + 4 * (lane_out >> 5);
      if (g.Of) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          store_part(g.Of + (int64_t)m * g.Nn + nb + 8 * q4,
                    make_float4(acc[a][b][4 * q4], acc[a][b][4 * q4 + 1], acc[a][b][4 * q4 + 2], acc[a][b][4 * q4 + 3]));
      }
      if (g.Oq) {
        const double inv = PIECES == 1 ? inv_out : read_lane_f64(inv_out, value_lane<PIECES>(a / PM * PIECES_N + b / PN));
        // Codes go to LDS first, laid out as the TM x TN byte tile with its 16-byte chunks XOR-swizzled by the
        // row, so that the tile can be written to memory as whole rows.
        const int row = 32 * (wm0 + a) + (lane_out & 31);
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int col = 32 * (wn0 + b) + 8 * q4 + 4 * (lane_out >> 5);
          const int chunk = (col >> 4) ^ (row & (TN / 16 - 1));
          *reinterpret_cast<uint32_t*>(code_row(row) + 16 * chunk + (col & 15)) =
              quantize4(acc[a][b][4 * q4], acc[a][b][4 * q4 + 1], acc[a][b][4 * q4 + 2], acc[a][b][4 * q4 + 3], inv);
        }
      }
    }
  if (g.Oq) {
    // TN / 16 consecutive lanes write one TN-byte row of the tile: full 128-byte lines for the 128-wide tile.
    __syncthreads();
    constexpr int CPRO = TN / 16;
    static_assert((TM * CPRO) % (64 * NW) == 0, "whole passes over the code tile");
#pragma unroll
    for (int i = 0; i < (TM * CPRO) / (64 * NW); ++i) {
      const int id = i * 64 * NW + tid_out;
      const int row = id / CPRO, c = id % CPRO;
      if (m0 + row < g.M && n0 + 16 * c < g.Nn) {
        const uint4 v = *reinterpret_cast<const uint4*>(code_row(row) + 16 * (c ^ (row & (CPRO - 1))));
        store_out(g.Oq + (int64_t)(m0 + row) * g.Nn + n0 + 16 * c, v);
      }
    }
  }
}

// A product's tile function with its compile-time shape, for the kernels below.
template <int B, int WM, int WN, int WGM, int WGN, bool AK, bool BK, bool DUMP = false>
struct GemmInstance {
  typedef GemmShape<B, WM, WN, WGM, WGN, AK, BK> Shape;
  static constexpr int BLOCK = B;
  static constexpr bool A_KMAJOR = AK, B_KMAJOR = BK;
  // Resident waves per SIMD the register allocation has to allow.  Four waves: 3 for the 128x128 tile and for the 64x64
  // tile at B = 64 (three workgroups share the LDS of a compute unit), else 4.  Eight waves: 4 for the 256x128 tile and 6 for
  // the 128x64 tile at B = 32 (two and three workgroups per compute unit), else 2 (one).
  static constexpr int WMIN = Shape::NW == 8 ? (B == 32 ? (WM * WN == 1 ? 6 : 4) : 2) : (WM * WN == 4 || B == 64) ? 3 : 4;
  template <class LATE>
  static __device__ __forceinline__ void run(const GemmArgs& g, int tile_index, int ntiles, int8_t* s_ring, float (*s_amax)[8], LATE&& late) {
    gemm_tile<B, WM, WN, WGM, WGN, AK, BK, DUMP>(g, tile_index, ntiles, s_ring, s_amax, late);
  }
};

// ---- Kernel arguments: operands and sizes first, all that the first stage's loads need (strides are computed), the rest read behind
// those loads (see kernel_arguments_from_here); the structures below are what the argument segment holds, the kernels' parameters in order.
struct GemmResults {   // as in GemmArgs
  int8_t* Oq;
  float *Os, *Of;
  int32_t* dump;
  int dump_kb;
};
typedef unsigned long long v2u64 __attribute__((ext_vector_type(2)));
struct GemmKernelArgs {   // few and wide, each costs the host 0.01 us of a launch (256^3 back to back 4.00 us; as nine up to 4.14)
  v2u64 operands, scales;
  v4i sizes;
  GemmResults results;
};
struct GemmPairKernelArgs {
  v2u64 dY_W;
  v4i sizes, deal;
  const int8_t* X;
  v2u64 SdY_SW;
  const float* SX;
  GemmResults dgrad, wgrad;
};
__device__ __forceinline__ void set_results(GemmArgs& g, const __attribute__((address_space(4))) GemmResults& r) {
  g.Oq = r.Oq, g.Os = r.Os, g.Of = r.Of, g.dump = r.dump, g.dump_kb = r.dump_kb;
}
template <class P>
__device__ __forceinline__ GemmArgs operands(const int8_t* A, const int8_t* Bm, const float* SA, const float* SB, int M, int Nn, int K) {
  GemmArgs g{A, Bm, SA, SB, M, Nn, K, 0, 0, 0, 0, 0, 0, nullptr, nullptr, nullptr, nullptr, 0};
  g.set_strides(P::BLOCK, P::A_KMAJOR, P::B_KMAJOR);
  return g;
}
template <class P>
__host__ __device__ __forceinline__ int tiles_of(int M, int Nn) {
  return (int)((unsigned)(M + P::Shape::TM - 1) / P::Shape::TM * ((unsigned)(Nn + P::Shape::TN - 1) / P::Shape::TN));
}

// One product per launch.
template <class P>
__global__ void __launch_bounds__(64 * P::Shape::NW, P::WMIN) gemm_kernel(const v2u64 pointers, const v2u64 scales, const v4i sizes, const GemmResults) {
  __shared__ __align__(1024) int8_t s_ring[P::Shape::LDS_BYTES];
  __shared__ float s_amax[8][8];
  P::run(operands<P>((const int8_t*)pointers[0], (const int8_t*)pointers[1], (const float*)scales[0], (const float*)scales[1], sizes[0], sizes[1], sizes[2]),
         blockIdx.x, sizes[3], s_ring, s_amax,
         [](GemmArgs& g) __attribute__((always_inline)) { set_results(g, kernel_arguments_from_here<GemmKernelArgs>()->results); });
}

// How the tiles of two products are dealt to the workgroups of one launch.  Numbers below `split` are tiles of the product that goes first,
// the one with the larger K times tile, the rest the other's; both counts are rounded up to multiples of 8, so that tile i is on XCD i % 8 (what exceeds a
// product's tiles is idle).  few == 0: in that order.  A launch of which all workgroups are resident at once puts workgroups b, b + 256, ...
// on one compute unit (measured: of 672 and 768 workgroups all), some units with one more than the `few` others.  Dealt in order,
// units come to have one more tile and more of the long ones as well; instead the `few` get `few_long` of the first product's, by turns, and
// the units with one more the rest.
struct PairDeal {
  int split, few, few_long, few_slots;   // few_slots: workgroups on the units that have one less
  // the tile of workgroup `index`: of the product that goes first?
  __host__ __device__ bool place(int index, int& tile) const {
    if (few == 0) {
      tile = index < split ? index : index - split;
      return index < split;
    }
    const int unit = index % 256, turn = index / 256, many = 256 - few;
    const int slot = unit >= many ? turn * few + unit - many : turn * many + unit, longs = unit >= many ? few_long : split - few_long;
    if (slot < longs) tile = unit >= many ? slot : few_long + slot;
    else tile = unit >= many ? slot - longs : few_slots - few_long + slot - longs;
    return slot < longs;
  }
};
// Both products of a layer in one launch: on which tiles (numbered as in jf_gemm_shapes.hpp; 0: in two launches), whether the second, the
// weight gradient, goes first, and how they are dealt.
struct PairChoice {
  int pair;
  bool second_first;
  PairDeal deal;
};
// `first`, `second`: tiles of the products in the order of the launch; work: what a tile of each takes, by the estimate that the choice
// among the pairs goes by, so that the launch is dealt as the choice counts on; resident: workgroups of a unit.  *most: the work of the
// busiest unit.  (672 tiles of 4096 x 768 -> 3072, of work 4 and 3: at most 10 on a unit instead of 11, 47.5 -> 45.3 us.)
// By K times the tile's size instead, which for 32x32 beside 64x64 tiles is far from their times, 3008 x 192 -> 960 took 14.1 us, in order
// 11.2, so 10.2; 6016 x 160 -> 1536 37.0, 21.5 and 20.0.
// Dealt where that unit has less to do than in order: 777 pairs of random layers both ways, 3 % less time in the mean, and where the model
// promises less than 7 % still 1 (to ask for those 7 % changed 880 layers by 0.1 %).
inline PairDeal deal_pair(int first, int second, double first_work, double second_work, int resident, double* most) {
  PairDeal d = {(first + 7) & ~7, 0, 0, 0};
  const int all = d.split + ((second + 7) & ~7), turns = all / 256, many = all % 256, few = 256 - many;
  // in order the unit with most is the first or the last of the first product's last round, or the first of the second's
  double least = 0.0;
  for (const int i : {0, d.split % 256, (first - 1) % 256}) {
    const int j = (i - d.split % 256 + 256) % 256;
    const int n1 = i < first ? (first - i + 255) / 256 : 0, n2 = j < second ? (second - j + 255) / 256 : 0;
    least = std::max(least, n1 * first_work + n2 * second_work);
  }
  if (all > 256 && all <= 256 * (int64_t)resident && many > 0) {
    // `units` with `slots` workgroups each and `there` of the first product's among them by turns: the most that one has (its tiles may be the shorter ones)
    const auto most_of = [&](int units, int slots, int there) {
      const auto work = [&](int n) { return n * first_work + (slots - n) * second_work; };
      return std::max(work(there / units), work((there + units - 1) / units));
    };
    for (int n = 0; n <= turns; ++n) {   // tiles of the first product on the units with fewer
      const int there = std::min(d.split, n * few), rest = d.split - there;
      if (rest > many * (turns + 1)) continue;
      const double busiest = std::max(most_of(few, turns, there), most_of(many, turns + 1, rest));
      if (busiest < least) least = busiest, d.few = few, d.few_long = there, d.few_slots = turns * few;
    }
  }
  *most = least;
  return d;
}

// Two independent products in one launch -- the input gradient and the weight gradient of a layer (Sec. 4), which
// need the same dY and nothing of each other.  Each product alone leaves compute units idle in its last round of tiles
// and pays its own ramp-up, first-stage latency and epilogue; in one launch the scheduler starts tiles of the second as
// those of the first finish, so that those phases of some workgroups run beside the K loops of others.
// (second_first: the second product's tiles are the longer ones.)
template <class P1, class P2>
__global__ void __launch_bounds__(64 * P1::Shape::NW, (P1::WMIN < P2::WMIN ? P1::WMIN : P2::WMIN))
gemm_pair_kernel(const v2u64 dY_W, const v4i sizes, const v4i deal, const int8_t* X, const v2u64, const float*, const GemmResults, const GemmResults) {
  static_assert(P1::Shape::NW == P2::Shape::NW, "one workgroup size");
  constexpr int LDS = P1::Shape::LDS_BYTES > P2::Shape::LDS_BYTES ? P1::Shape::LDS_BYTES : P2::Shape::LDS_BYTES;
  __shared__ __align__(1024) int8_t s_ring[LDS];
  __shared__ float s_amax[8][8];
  const int8_t *const dY = (const int8_t*)dY_W[0], *const W = (const int8_t*)dY_W[1];
  const int N = sizes[0], C = sizes[1], D = sizes[2], second_first = sizes[3];
  int i;
  const bool early = PairDeal{deal[0], deal[1], deal[2], deal[3]}.place(blockIdx.x, i);
  if (early != (second_first != 0)) {
    const int tiles = tiles_of<P1>(N, C);
    if (i < tiles)
      P1::run(operands<P1>(dY, W, nullptr, nullptr, N, C, D), i, tiles, s_ring, s_amax, [](GemmArgs& g) __attribute__((always_inline)) {
        const auto a = kernel_arguments_from_here<GemmPairKernelArgs>();
        g.SA = (const float*)a->SdY_SW[0], g.SB = (const float*)a->SdY_SW[1];
        set_results(g, a->dgrad);
      });
  } else {
    const int tiles = tiles_of<P2>(D, C);
    if (i < tiles)
      P2::run(operands<P2>(dY, X, nullptr, nullptr, D, C, N), i, tiles, s_ring, s_amax, [](GemmArgs& g) __attribute__((always_inline)) {
        const auto a = kernel_arguments_from_here<GemmPairKernelArgs>();
        g.SA = (const float*)a->SdY_SW[0], g.SB = a->SX;
        set_results(g, a->wgrad);
      });
  }
}

// --------------------------------------------------------------------- host
inline GemmResults results_of(const GemmArgs& a) { return {a.Oq, a.Os, a.Of, a.dump, a.dump_kb}; }
template <class P>
static void launch_one(const GemmArgs& a, hipStream_t st) {
  typedef KernelParameters<decltype(&gemm_kernel<P>)> Parameters;
  static_assert(Parameters::template preloaded<2>() && Parameters::template stands_at<3, GemmResults>(offsetof(GemmKernelArgs, results)), "GemmKernelArgs");
  const int tiles = tiles_of<P>(a.M, a.Nn);
  const v2u64 pointers = {(unsigned long long)a.A, (unsigned long long)a.Bm}, scales = {(unsigned long long)a.SA, (unsigned long long)a.SB};
  hipLaunchKernelGGL((gemm_kernel<P>), dim3(tiles), dim3(64 * P::Shape::NW), 0, st, pointers, scales, v4i{a.M, a.Nn, a.K, tiles}, results_of(a));
}
// input gradient (first) and weight gradient
template <class P1, class P2>
static void launch_pair(const GemmArgs& a1, const GemmArgs& a2, const PairChoice& choice, hipStream_t st) {
  typedef GemmPairKernelArgs Args;
  typedef KernelParameters<decltype(&gemm_pair_kernel<P1, P2>)> Parameters;
  static_assert(Parameters::template preloaded<3>() && Parameters::template stands_at<4, v2u64>(offsetof(Args, SdY_SW)) &&
                    Parameters::template stands_at<5, const float*>(offsetof(Args, SX)) && Parameters::template stands_at<6, GemmResults>(offsetof(Args, dgrad)) &&
                    Parameters::template stands_at<7, GemmResults>(offsetof(Args, wgrad)), "GemmPairKernelArgs");
  const PairDeal& deal = choice.deal;
  const int all = deal.split + (((choice.second_first ? tiles_of<P1>(a1.M, a1.Nn) : tiles_of<P2>(a2.M, a2.Nn)) + 7) & ~7);
  const v2u64 dY_W = {(unsigned long long)a1.A, (unsigned long long)a1.Bm}, SdY_SW = {(unsigned long long)a1.SA, (unsigned long long)a1.SB};
  hipLaunchKernelGGL((gemm_pair_kernel<P1, P2>), dim3(all), dim3(64 * P1::Shape::NW), 0, st, dY_W, v4i{a1.M, a1.Nn, a1.K, (int)choice.second_first},
                     v4i{deal.split, deal.few, deal.few_long, deal.few_slots}, a2.Bm, SdY_SW, a2.SB, results_of(a1), results_of(a2));
}

template <bool AK, bool BK>
struct FineInstance;   // jf_gemm_fine.hpp
template <int B, bool AK, bool BK>
static void launch_wide(const GemmArgs& a, hipStream_t st);   // jf_gemm_wide.hpp

// Launches the product on tile shape `shape`, numbered and chosen as jf_gemm_shapes.hpp says.  One translation unit per
// (product, block size) instantiates this, so that the kernels compile in parallel.  AK / BK: operand A / Bm is K-major.
template <int B, bool AK, bool BK, bool DUMP>
static void launch_shape(int shape, const GemmArgs& a, hipStream_t st) {
  if constexpr (B > 32 && !DUMP) {
    if (shape == 11) return launch_wide<B, AK, BK>(a, st);
  }
  if constexpr (B == 128) {
    if (shape == 6) launch_one<GemmInstance<B, 2, 2, 4, 2, AK, BK, DUMP>>(a, st);
    else launch_one<GemmInstance<B, 2, 1, 2, 4, AK, BK, DUMP>>(a, st);
  } else {
    if (shape == 1) launch_one<GemmInstance<B, 2, 2, 2, 2, AK, BK, DUMP>>(a, st);
    else if constexpr (B == 32) {
      if (shape == 6) launch_one<GemmInstance<B, 2, 2, 4, 2, AK, BK, DUMP>>(a, st);
      else if (shape == 8) launch_one<GemmInstance<B, 2, 1, 2, 2, AK, BK, DUMP>>(a, st);
      else if (shape == 7) launch_one<GemmInstance<B, 1, 1, 4, 2, AK, BK, DUMP>>(a, st);
      else if (DUMP || shape == 4) launch_one<GemmInstance<B, 1, 1, 2, 2, AK, BK, DUMP>>(a, st);
      else launch_one<FineInstance<AK, BK>>(a, st);
    } else {
      launch_one<GemmInstance<B, 1, 1, 2, 2, AK, BK, DUMP>>(a, st);
    }
  }
}
template <int B, bool AK, bool BK>
static void launch_product(int shape, const GemmArgs& a, bool dump, hipStream_t st) {
  if (dump) launch_shape<B, AK, BK, true>(shape, a, st);
  else launch_shape<B, AK, BK, false>(shape, a, st);
}

#define JF_GEMM_INSTANCE(NAME, B, AK, BK) \
  namespace jf { void NAME(int shape, const GemmArgs& a, bool dump, hipStream_t st) { launch_product<B, AK, BK>(shape, a, dump, st); } }

}  // namespace jf
