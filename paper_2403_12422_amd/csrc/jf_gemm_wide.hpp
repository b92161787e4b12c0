// Persistent 256x256 form of the products at block sizes 64 and 128 (jf_gemm_kernel.hpp) for outputs of many tiles.
//
// What bounds these products is what moves the operands: at 8192^3 and block 128 the kernel without its loads and fragment reads
// takes 427 of 527 us, and the chip, which lowers its clock under this load (to 1.7-1.9 GHz), gives back in clock what a
// shorter loop saves, so that bytes moved per MFMA count for more than instructions.  A 256x256 tile takes a third less out of
// L2 than 256x128, and a wave that owns 64x128 outputs a quarter less out of LDS than one of 64x64.  Eight waves, two per SIMD,
// have 256 registers each: 128 accumulators, two INT32 tiles, one set of fragments.
// One workgroup owns a compute unit, so nothing runs beside the start and the end of a tile.  The workgroups are therefore
// persistent: the stages of all tiles of a workgroup are one stream of loads, which runs on through the epilogue, and the
// pipeline reads the first fragments of the next tile beside the last folds of this one.
// Measured, forward / dgrad / wgrad in us, against the best tile of jf_gemm_kernel.hpp:
//   block 128  8192^3           593 / 594 / 598 -> 528 / 533 / 531      16384 x 4096 -> 11008  876 / 787 / 840 -> 734 / 712 / 731
//   block 128  4096^3           79.5 / 80.2 / 80.7 -> 72.0 / 72.8 / 72.6
//   block 64   8192^3           764 / 738 / 722 -> 708 / 687 / 725      4096^3  102.5 / 100.0 / 98.3 -> 92.6 / 91.4 / 90.5
// and less since, by the priorities in run_stage and the instruction that wide_quarters chooses (8192^3 at block 128 forward 541 -> 514).
// (At block 64 the vector ALU bounds the loop, for which two waves per SIMD do a little worse than three: what is gained is the
// start and end of the tiles, and it is lost again where 256x256 tiles fill the compute units unevenly.)
#pragma once
#include "jf_gemm_kernel.hpp"

namespace jf {

template <int B, bool AK, bool BK>
struct WideShape {
  // A stage is one quantization block of K: 64 KB at B = 128, of which two fit the LDS; four of 32 KB at B = 64.
  static constexpr int KC = B, NBUF = B == 128 ? 2 : 4, NW = 8, TM = 256, TN = 256;
  static constexpr int WM = 2, WN = 4;   // 32x32 sub-blocks of a wave; the waves stand 4 x 2
  static constexpr int A_BYTES = TM * KC, B_BYTES = TN * KC;
  // The ring holds the stages of A and behind them those of Bm, so that every LDS read reaches its stage by the 16-bit offset
  // of the instruction.
  static constexpr int RING_A = NBUF * A_BYTES, LDS_BYTES = RING_A + NBUF * B_BYTES;
  static_assert(RING_A <= 65536 && LDS_BYTES - RING_A <= 65536, "16-bit offsets");
};

// A wave's MFMA on the sub-blocks of a 256x256 tile: v_mfma_i32_32x32x32_i8, or, QUARTERS, v_mfma_i32_16x16x64_i8 on their quarters.  Both
// take 16 bytes of K per lane and the same matrix cycles per multiply-add.  The latter writes its INT32 tile, and reads it in a chain, half
// as often, which is power, what bounds large products at B = 128, at the price of twice the instructions to issue: bare chains of
// random codes with their folds 24.9 -> 23.7 ns per 32x32x32, of zeros, at full clock, 18.5 -> 20.9.  8192^3 at B = 128 forward 536 -> 513
// us, 16384 x 4096 -> 11008 forward 741 -> 720, input gradient 714 -> 694; where both operands are read transposed, by twice the LDS
// instructions, it loses (weight gradient 734 -> 742), and at B = 64 the bare chains do (33.4 -> 34.9).
// Where units are left idle the others run at a higher clock, and what counts is the instructions.  Quarters and whole sub-blocks by tiles,
// 256 at a time on the units, K = 4096, in us: forward 64 tiles 56.3 and 49.3, 128 56.9 and 49.9, 160 57.5 and 53.2, 176 57.9 and 56.1, 192 59.1 and 58.3, 208 61.7
// and 62.2, 224 63.8 and 65.3, 256 68.5 and 70.0, 320 116.0 and 112.3, 384 116.8 and 115.8; input gradient, K = 2048, 160 34.1 and 31.2, 256 39.5
// and 40.4, 272 64.7 and 62.3, 400 45.9 and 45.5, 448 equal, 480 71.4 and 73.4.  The line: four fifths of the rounds' places taken.
inline bool wide_quarters(int64_t tiles) { return 5 * tiles >= 4 * 256 * ((tiles + 255) / 256); }
constexpr int wide_fragment_rows(bool quarters) { return quarters ? 16 : 32; }   // its 64 lanes hold 1 KB either way

// LDS addresses of an operand's fragments: as FragAddr, of whose offsets every one is the first with bits of the chunk number
// toggled, so that a lane keeps one address per operand.  Fragment j of a sub-tile: K step j of 32 bytes, or, of 16 rows, the half
// j % 2 of the rows and 64 bytes of K from 64 (j / 2) on.
template <int TILE, bool KMAJOR, int KC, int ROWS>
struct WideFrag {
  typedef TileLayout<TILE, KMAJOR, KC> L;
  uint32_t at;
  __device__ __forceinline__ void init(const int8_t* ring, int region, int sub0, int lane) {
    int first;
    if (KMAJOR) {
      first = 16 * L::slot(sub0 * 32 + lane % ROWS, lane / ROWS);
    } else {   // transposing reads, see FragAddr
      const int i = lane & 15, g = lane >> 4;
      first = 16 * L::slot(16 * (ROWS == 32 ? g >> 1 : g) + (i >> 1), sub0 * 2 + (ROWS == 32 ? g & 1 : 0)) + 8 * (i & 1);
    }
    at = (uint32_t)(uintptr_t)(lds_ptr)(ring) + (uint32_t)(region + first);
  }
  // fragment j of sub-tile u (relative to the wave's first), of the stage `stage` bytes into the region
  __device__ __forceinline__ v4i read(int stage, int u, int j) const {
    const int k = ROWS == 32 ? 32 * j : 64 * (j >> 1), half = ROWS == 32 ? 0 : j & 1;   // first byte of K, rows 16 half on
    if (KMAJOR) {
      return *(lds_v4i)(uintptr_t)((at ^ k) + stage + (u * 32 + half * 16) * (L::kCPR * 16));
    } else {
      const uint32_t p = (at ^ (32 * u + 16 * half)) + stage + k * (L::kCPR * 16);
      const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(uintptr_t)(p));
      const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(uintptr_t)(p + 8 * L::kCPR * 16));
      return v4i{lo[0], lo[1], hi[0], hi[1]};
    }
  }
};

// One operand's side of the stream of stages, in direct-to-LDS loads.  Load n of a wave fills the 64 chunks from slot
// (n * NW + wave) * 64 on: the lane's share of its address depends neither on n nor on the stage (the swizzle repeats every 16
// rows at most), the rest is uniform.  Rows or columns outside the matrix are replaced by valid ones, as in chunk_offset; the
// rows of one load lie all inside or all outside, since they share a quantization block.
template <int TILE, bool KMAJOR, int KC, int NW>
struct WideLoads {
  typedef TileLayout<TILE, KMAJOR, KC> L;
  static constexpr int N = TILE * KC / (1024 * NW);   // loads per wave and stage
  static constexpr int ROWS = 64 / L::kCPR;           // LDS rows of one load
  uint32_t voff, soff[N];
  const int8_t* base;
  // the tile whose first element is `origin`; outer_left: from there to the matrix' edge
  __device__ __forceinline__ void set_tile(const int8_t* origin, int outer_left, uint32_t ld, int wave, int lane) {
    base = uniform_pointer(origin);
    const int r = lane / L::kCPR, c = (lane % L::kCPR) ^ L::swz(ROWS * wave + r);
    voff = (uint32_t)r * ld + (uint32_t)(KMAJOR ? 16 * c : min(16 * c, outer_left - 16));
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int row = (n * NW + wave) * ROWS;
      soff[n] = (KMAJOR && row >= outer_left ? 0u : (uint32_t)row) * ld;
    }
  }
  // load n into the stage BYTE bytes from `lds`, the LDS address of the wave's first chunk in the ring
  template <int BYTE>
  __device__ __forceinline__ void issue(int n, uint32_t lds) const {
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(base + soff[n]), "s"(lds), "n"(BYTE)
                 : "memory", "m0", "scc");
  }
};

// A product's arguments where the kernel finds them.  They are read again wherever a tile begins or ends: kept in scalar
// registers throughout they push each other, and with them vector registers, out of the K loop.
typedef const __attribute__((address_space(4))) GemmArgs* KernelArgs;
__device__ __forceinline__ KernelArgs read_again(KernelArgs a) {
  asm volatile("" : "+s"(a));
  return a;
}

// Tiles tile_index, tile_index + stride, ... of `ntiles`, on a workgroup of eight waves; tile_index < ntiles.
template <int B, bool AK, bool BK, bool QUARTERS>
__device__ __forceinline__ void gemm_wide(const KernelArgs args, const int wave, int tile_index, const int stride, const int ntiles,
                                          int8_t* const s_ring, float* const s_amax) {
  typedef WideShape<B, AK, BK> S;
  constexpr int KC = S::KC, NBUF = S::NBUF, NW = S::NW, TM = S::TM, TN = S::TN, WM = S::WM, WN = S::WN;
  constexpr int KPB = B / 32, NT = WM * WN;   // MFMAs of a unit (sub-block x K block), units of a stage
  constexpr int NSB = WN * 32 / B;            // block columns of a wave
  static_assert(WM * 32 <= B && NSB >= 1, "a wave has one block row and whole block columns");

  const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN;   // first sub-block of this wave inside the tile
  const int nstages = args->K / KC;

  // tiles to XCDs as in gemm_tile (stride is a multiple of 8 wherever a workgroup has several tiles)
  constexpr int GROUP_M = 4;
  auto origin_of = [&](int index, int& m0, int& n0) __attribute__((always_inline)) {
    const KernelArgs g = read_again(args);
    const int tiles_n = (g->Nn + TN - 1) / TN, tiles_m = (g->M + TM - 1) / TM;
    const int xcd = index & 7, idx = index >> 3;
    const int tile = xcd * (ntiles >> 3) + min(xcd, ntiles & 7) + idx;
    const int group = tile / (GROUP_M * tiles_n), first_m = group * GROUP_M;
    const int in_group = tile - group * GROUP_M * tiles_n, group_rows = min(GROUP_M, tiles_m - first_m);
    m0 = (first_m + in_group % group_rows) * TM;
    n0 = (in_group / group_rows) * TN;
  };
  // the tile after `index` (the last one again when there is none: its addresses are valid, what they deliver is not used)
  auto following = [&](int index) __attribute__((always_inline)) { return index + stride < ntiles ? index + stride : index; };

  // ---- the stream of stages
  WideLoads<TM, AK, KC, NW> loadA;
  WideLoads<TN, BK, KC, NW> loadB;
  constexpr int LOADS_A = decltype(loadA)::N, LOADS = LOADS_A + decltype(loadB)::N;
  const int64_t kstepA = AK ? KC : KC * args->lda, kstepB = BK ? KC : KC * args->ldb;
  const uint32_t lds_wave = lds_address(s_ring, 1024 * wave);
  int load_index = tile_index, load_left;
  auto set_loads = [&]() __attribute__((always_inline)) {
    const KernelArgs g = read_again(args);
    int m, n;
    origin_of(load_index, m, n);
    const int lane = lane_again();
    loadA.set_tile(g->A + (AK ? (int64_t)m * g->lda : (int64_t)m), g->M - m, (uint32_t)g->lda, wave, lane);
    loadB.set_tile(g->Bm + (BK ? (int64_t)n * g->ldb : (int64_t)n), g->Nn - n, (uint32_t)g->ldb, wave, lane);
    load_left = nstages;
  };
  auto issue_load = [&](auto slot_tag, auto n_tag) __attribute__((always_inline)) {   // load n of the stream's next stage
    constexpr int slot = decltype(slot_tag)::value, n = decltype(n_tag)::value;
    if constexpr (n < LOADS_A) loadA.template issue<slot * S::A_BYTES + 1024 * NW * n>(n, lds_wave);
    else loadB.template issue<S::RING_A + slot * S::B_BYTES + 1024 * NW * (n - LOADS_A)>(n - LOADS_A, lds_wave);
    if constexpr (n + 1 == LOADS) {
      loadA.base += kstepA;
      loadB.base += kstepB;
      if (--load_left == 0) {
        load_index = following(load_index);
        set_loads();
      }
    }
  };

  // ---- block scales, by scalar loads two stages ahead: one stage to arrive, one as a product
  typedef const __attribute__((address_space(4))) float* ScalePtr;
  ScalePtr scaleA, scaleB;
  const int sa_k = args->sa_k, sb_k = args->sb_k;
  int scale_index = tile_index, scale_left, scale_step;
  auto set_scales = [&]() __attribute__((always_inline)) {
    const KernelArgs g = read_again(args);
    int m, n;
    origin_of(scale_index, m, n);
    const int ra = min((m + 32 * wm0) / B, g->M / B - 1), rb = min((n + 32 * wn0) / B, g->Nn / B - 1);
    scaleA = (ScalePtr)uniform_pointer(g->SA + (int64_t)ra * g->sa_p);
    scaleB = (ScalePtr)uniform_pointer(g->SB + (int64_t)rb * g->sb_p);
    scale_step = rb + 1 < g->Nn / B ? g->sb_p : 0;
    scale_left = nstages;
  };
  float arriving_a, arriving_b[NSB], scale[NSB], scale_next[NSB];
  auto request_scales = [&]() __attribute__((always_inline)) {
    arriving_a = *scaleA;
#pragma unroll
    for (int k = 0; k < NSB; ++k) arriving_b[k] = scaleB[k * scale_step];
    scaleA += sa_k;
    scaleB += sb_k;
    if (--scale_left == 0) {
      scale_index = following(scale_index);
      set_scales();
    }
  };
  auto take_scales = [&](float (&s)[NSB]) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NSB; ++k)
      s[k] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, arriving_a * arriving_b[k])));
  };

  // ---- the pipeline of gemm_tile with one set of fragments: unit i of a stage is sub-block (i / WN, i % WN); the chain of unit
  // i + 1 is issued beside the fold of unit i.  A fragment is read into the registers that have just come out of use: those of
  // the second sub-block row beside unit WN - 2, behind the last chain of the first; those of the next stage beside the
  // units from SYNC on, which the barrier stands before.
  WideFrag<TM, AK, KC, wide_fragment_rows(QUARTERS)> fragA;
  WideFrag<TN, BK, KC, wide_fragment_rows(QUARTERS)> fragB;
  const int lane = lane_again();
  fragA.init(s_ring, 0, wm0, lane);
  fragB.init(s_ring, S::RING_A, wn0, lane);
  v4i fa[KPB], fb[WN][KPB];
  v16i vi[2];
  float acc[WM][WN][16];
  const v16i zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  auto read_a = [&](int slot, int a, int j) __attribute__((always_inline)) { fa[j] = fragA.read(slot * S::A_BYTES, a, j); };
  auto read_b = [&](int slot, int b, int j) __attribute__((always_inline)) { fb[b][j] = fragB.read(slot * S::B_BYTES, b, j); };
  // step js of the chain of unit i: an MFMA, or two, of the quarters (js % 2, 0) and (js % 2, 1) over half of K (part 0 and 1)
  auto chain_step = [&](int i, int js, int part, v16i& dst) __attribute__((always_inline)) {
    if constexpr (QUARTERS) {
      const int q = 2 * (js & 1) + part;
      const v4i c = js < 2 ? v4i{0, 0, 0, 0} : v4i{dst[4 * q], dst[4 * q + 1], dst[4 * q + 2], dst[4 * q + 3]};
      const v4i d = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[i % WN][(js & 2) + part], fa[js], c, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) dst[4 * q + r] = d[r];
    } else {
      dst = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[i % WN][js], fa[js], js == 0 ? zero16 : dst, 0, 0, 0);
    }
  };
  constexpr int PARTS = QUARTERS ? 2 : 1;   // MFMAs of a step; each has its share of the fold behind it
  constexpr bool PHASES = B == 64;          // but here all of it stands behind the last (see run_stage)
  static_assert(!PHASES || PARTS == 1, "whole sub-blocks");
  auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
      for (int b = 0; b < WN; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
  };
  // all but the youngest `left` loads of this wave have landed, and its LDS reads are done
  auto wait_loads = [&](auto left) __attribute__((always_inline)) {
    constexpr int N = decltype(left)::value;
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
  };
  auto meet = [&]() __attribute__((always_inline)) { asm volatile("s_barrier" ::: "memory"); };

  // stage in ring slot u; after_store: the stores of an epilogue may be outstanding, which are not counted in order with loads
  auto run_stage = [&](auto u_tag, bool after_store) __attribute__((always_inline)) {
    constexpr int slot = decltype(u_tag)::value, nslot = (slot + 1) % NBUF, SYNC = WN;
    // The toggled addresses are formed again in each stage: kept over the loop they go to scratch memory, for whose loads the stages in
    // flight are waited for.
    if constexpr (B == 128 && AK && !(BK && QUARTERS)) asm volatile("" : "+v"(fragB.at));
    static_for<0, NT>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value, a = i / WN, b = i % WN;
      v16i &cur = vi[i & 1], &nxt = vi[(i & 1) ^ 1];
      // The arbiter favours the older of a SIMD's two waves, which then waits at the barrier while the other, alone, leaves the pipes
      // idle.  Between two barriers the wave that is behind goes first (16384 x 4096 -> 11008 at B = 128 759 / 732 / 749 -> 741 / 715 /
      // 734 us forward / dgrad / wgrad, both gradients 1488 -> 1450; 4096^3 at B = 64 93.2 / 92.5 / 91.9 -> 92.8 / 91.4 / 89.7).
      // PHASES (B = 64, where the vector ALU bounds the loop): conversions issue at 4.3 cycles and FMAs at 2.3, and those of two waves run beside each
      // other.  Left alone both waves convert and then both add.  So all of a unit's conversions stand before its FMAs, and a wave in its FMAs and the
      // next chain goes before one in its conversions: bare chains of 2 MFMAs with their folds, two waves, random codes 36.6 -> 29.5 ns
      // per MFMA, small numbers 31.3 -> 25.0; 8192^3 683 / 670 / 665 -> 671 / 649 / 644 us, 4096^3 91.2 -> 90.0, both gradients 177.6 -> 172.5.
      // (At B = 128 the fold is too short for it: 16384 x 4096 -> 11008 1390 -> 1400.  At B = 32, four waves of two workgroups to a SIMD, bare chains
      // gain 10-20 %, the kernels lose 1-2: there the power limit and the fragments' way into the registers bound the loop.)
      constexpr int since = (i - SYNC + NT) % NT, LOW = since < NT / 2 ? 2 : 0;
      if constexpr (!PHASES && i % 2 == 0) __builtin_amdgcn_s_setprio(3 - since / 2);
      if constexpr (i == SYNC) {
        if (NBUF > 2 && !after_store) wait_loads(std::integral_constant<int, LOADS * (NBUF - 2)>());
        else wait_loads(std::integral_constant<int, 0>());
        meet();
        take_scales(scale_next);
        request_scales();
      }
      static_for<0, KPB>([&](auto js_tag) __attribute__((always_inline)) {
        constexpr int js = decltype(js_tag)::value;
        chain_step((i + 1) % NT, js, 0, nxt);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PHASES && js == KPB - 1) {
          __builtin_amdgcn_s_setprio(LOW);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (PARTS == 1 && i == WN - 2) read_a(slot, 1, js);
        if constexpr (PARTS == 1 && i == 2 * WN - 2) read_a(nslot, 0, js);
        if constexpr (i >= SYNC) {
          read_b(nslot, i - SYNC, js);
          // the loads of the stage NBUF ahead, into the slot of which every wave has read the last fragment
          constexpr int P = (NT - SYNC) * KPB, at = (i - SYNC) * KPB + js;
          static_for<0, LOADS>([&](auto n) __attribute__((always_inline)) {
            if constexpr (decltype(n)::value * P / LOADS == at) issue_load(u_tag, n);
          });
        }
        constexpr int R0 = 16 * js / KPB, R1 = 16 * (js + 1) / KPB, RM = QUARTERS ? (R0 + R1) / 2 : R1;
        if constexpr (!PHASES) {
          fold<R0, RM>(acc[a][b], cur, scale[b * NSB / WN]);
        } else if constexpr (js == KPB - 1) {
          float c[16];
          fold_convert(c, cur);
          __builtin_amdgcn_sched_barrier(0);
          __builtin_amdgcn_s_setprio(LOW + 1);
          __builtin_amdgcn_sched_barrier(0);
          fold_add(acc[a][b], c, scale[b * NSB / WN]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PARTS == 2) {
          chain_step((i + 1) % NT, js, 1, nxt);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (i == WN - 2) read_a(slot, 1, js);
          if constexpr (i == 2 * WN - 2) read_a(nslot, 0, js);
          fold<RM, R1>(acc[a][b], cur, scale[b * NSB / WN]);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    });
#pragma unroll
    for (int k = 0; k < NSB; ++k) scale[k] = scale_next[k];
  };

  // ---- epilogue: optional FP32 store, max-abs of the blocks, Eq. 1, codes.  Nothing goes through LDS, which holds the next
  // tile's first stages: lane l and l + 32 of a row hold its even and odd dwords, and after two half-wave swaps 16 consecutive
  // bytes each.  A wave has whole 128-byte lines, but 32 bytes of each per store: written back, so that L2 puts them
  // together (written through, 8192^3 at block 128 takes 560 instead of 549 us, 16384 x 4096 -> 11008 802 instead of 766).
  auto store_tile = [&](int m0, int n0) __attribute__((always_inline)) {
    const KernelArgs g = read_again(args);
    const int lane = lane_again();
    float amax[NSB];
#pragma unroll
    for (int k = 0; k < NSB; ++k) {
      float m = 0.0f;
#pragma unroll
      for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = k * (WN / NSB); b < (k + 1) * (WN / NSB); ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) m = fmaxf(m, fabsf(acc[a][b][r]));
      amax[k] = wave_group_max<63>(m);
    }
    if (B == 128) {   // two waves, one above the other, share a block
      if (lane == 0) s_amax[wave] = amax[0];
      __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));   // lgkmcnt 0; loads stay in flight
      meet();
      amax[0] = fmaxf(amax[0], s_amax[wave ^ 2]);
    }
    const int mrow0 = m0 + 32 * wm0, h = lane >> 5, g4 = lane >> 4;
    const int first_row = QUARTERS ? lane & 15 : lane & 31;
    if (mrow0 >= g->M) return;   // wave-uniform, as the skipped columns below
#pragma unroll
    for (int k = 0; k < NSB; ++k) {
      const int ncol0 = n0 + 32 * wn0 + k * B;
      if (ncol0 >= g->Nn) continue;
      float s;
      double inv;
      block_scale(amax[k], s, inv);
      if (g->Oq && lane == 0 && mrow0 % B == 0) store_part(&g->Os[(int64_t)(mrow0 / B) * (g->Nn / B) + ncol0 / B], s);
#pragma unroll
      for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN / NSB; ++b) {
          const float(&v)[16] = acc[a][k * (WN / NSB) + b];
          // Quad q holds columns 8 q + 4 h on of row lane % 32, or 16 (q % 2) + 4 g4 on of row 16 (q / 2) + lane % 16.
          const int64_t at = (int64_t)(mrow0 + 32 * a + first_row) * g->Nn + ncol0 + 32 * b;
          if (g->Of) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              store_part(g->Of + at + (QUARTERS ? (int64_t)16 * (q >> 1) * g->Nn + 16 * (q & 1) + 4 * g4 : 8 * q + 4 * h),
                         make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]));
          }
          if (g->Oq) {
            uint32_t c[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = quantize4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3], inv);
            const auto even = __builtin_amdgcn_permlane32_swap(c[0], c[2], false, false);
            const auto odd = __builtin_amdgcn_permlane32_swap(c[1], c[3], false, false);
            if constexpr (QUARTERS) {   // rows of lanes too: a lane ends with the 16 bytes of quarter g4
              const auto lo = __builtin_amdgcn_permlane16_swap(even[0], odd[0], false, false);
              const auto hi = __builtin_amdgcn_permlane16_swap(even[1], odd[1], false, false);
              store_part(g->Oq + at + (int64_t)16 * (g4 >> 1) * g->Nn + 16 * (g4 & 1), v4i{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]});
            } else {
              store_part(g->Oq + at + 16 * h, v4i{(int)even[0], (int)even[1], (int)odd[0], (int)odd[1]});
            }
          }
        }
    }
  };

  set_loads();
  set_scales();
  static_for<0, NBUF>([&](auto slot) __attribute__((always_inline)) {
    static_for<0, LOADS>([&](auto n) __attribute__((always_inline)) { issue_load(slot, n); });
  });
  request_scales();
  take_scales(scale);
  request_scales();
  zero_acc();
  wait_loads(std::integral_constant<int, LOADS * (NBUF - 1)>());
  meet();
  static_for<0, KPB>([&](auto j) __attribute__((always_inline)) {
    read_a(0, 0, decltype(j)::value);
    static_for<0, WN>([&](auto b) __attribute__((always_inline)) { read_b(0, decltype(b)::value, decltype(j)::value); });
  });
  static_for<0, KPB * PARTS>([&](auto n) __attribute__((always_inline)) {
    chain_step(0, decltype(n)::value / PARTS, decltype(n)::value % PARTS, vi[0]);
  });

  // passes over the ring; a tile begins at the slot behind the last stage of the tile before it
  bool stored = false;
  int t = 0, first_slot = 0;
#pragma unroll 1
  for (;;) {
    static_for<0, NBUF>([&](auto u) __attribute__((always_inline)) {
      if (decltype(u)::value >= first_slot && t < nstages) {
        run_stage(u, t == 0 && stored);
        ++t;
        if (t == nstages) first_slot = (decltype(u)::value + 1) % NBUF;
      }
    });
    if (t < nstages) {
      first_slot = 0;
      continue;
    }
    int m0, n0;
    origin_of(tile_index, m0, n0);
    store_tile(m0, n0);
    stored = true;
    tile_index += stride;
    if (tile_index >= ntiles) break;
    zero_acc();
    t = 0;
  }
  wait_loads(std::integral_constant<int, 0>());   // nothing may land in the ring any more
}

static constexpr int kWideWorkgroups = 256;   // one per compute unit: the ring takes 128 of its 160 KB of LDS

// One product per launch.  The arguments are read through the kernel's argument segment (see KernelArgs).
template <int B, bool AK, bool BK, bool QUARTERS>
__global__ void __launch_bounds__(512, 2) gemm_wide_kernel(const GemmArgs, const int ntiles) {
  __shared__ __align__(1024) int8_t s_ring[WideShape<B, AK, BK>::LDS_BYTES];
  __shared__ float s_amax[8];
  gemm_wide<B, AK, BK, QUARTERS>((KernelArgs)__builtin_amdgcn_kernarg_segment_ptr(), __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), blockIdx.x, gridDim.x, ntiles, s_ring, s_amax);
}

// Both backward products of a layer in one launch, the one with the longer tiles first (`second_first`: the weight gradient).
// The workgroups go through the tiles of both as one list, so that only its end is uneven.  `split`: the tiles of the
// product that goes first, rounded up to a multiple of 8 as in gemm_pair_kernel.
template <int B>
__global__ void __launch_bounds__(512, 2) gemm_wide_pair_kernel(const GemmArgs, const GemmArgs, const int tiles1, const int tiles2, const int split,
                                                                const int second_first) {
  __shared__ __align__(1024) int8_t s_ring[WideShape<B, true, false>::LDS_BYTES];
  __shared__ float s_amax[8];
  const KernelArgs args = (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr();
  const int n = gridDim.x, i = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int behind = (n - split % n + i) % n;   // this workgroup's first tile of the product that comes second
#pragma unroll 1
  for (int turn = 0; turn < 2; ++turn) {
    const int first = turn == 0 ? i : behind;
    if ((turn == 0) != (second_first != 0)) {
      if (first < tiles1) gemm_wide<B, true, false, B == 128>(args, wave, first, n, tiles1, s_ring, s_amax);
    } else {
      if (first < tiles2) gemm_wide<B, false, false, false>(args + 1, wave, first, n, tiles2, s_ring, s_amax);
    }
    __syncthreads();   // the next product's loads may not land before every wave is through with this one's
  }
}

template <int B, bool AK, bool BK, bool QUARTERS>
static void launch_wide_as(const GemmArgs& a, int tiles, hipStream_t st) {
  static_assert(KernelParameters<decltype(&gemm_wide_kernel<B, AK, BK, QUARTERS>)>::template stands_at<0, GemmArgs>(0), "read as KernelArgs");
  hipLaunchKernelGGL((gemm_wide_kernel<B, AK, BK, QUARTERS>), dim3(tiles < kWideWorkgroups ? tiles : kWideWorkgroups), dim3(512), 0, st, a, tiles);
}
template <int B, bool AK, bool BK>
static void launch_wide(const GemmArgs& a, hipStream_t st) {
  const int tiles = ((a.M + 255) / 256) * ((a.Nn + 255) / 256);
  if constexpr (B == 128 && AK) {
    if (wide_quarters(tiles)) return launch_wide_as<B, AK, BK, true>(a, tiles, st);
  }
  launch_wide_as<B, AK, BK, false>(a, tiles, st);
}
template <int B>
static void launch_wide_pair(const GemmArgs& a1, const GemmArgs& a2, hipStream_t st) {
  const int t1 = ((a1.M + 255) / 256) * ((a1.Nn + 255) / 256), t2 = ((a2.M + 255) / 256) * ((a2.Nn + 255) / 256);
  const bool second_first = a2.K > a1.K;
  typedef KernelParameters<decltype(&gemm_wide_pair_kernel<B>)> Parameters;
  static_assert(Parameters::template stands_at<0, GemmArgs>(0) && Parameters::template stands_at<1, GemmArgs>(sizeof(GemmArgs)), "read as KernelArgs and the next");
  const int split = ((second_first ? t2 : t1) + 7) & ~7, all = split + (second_first ? t1 : t2);
  hipLaunchKernelGGL((gemm_wide_pair_kernel<B>), dim3(all < kWideWorkgroups ? all : kWideWorkgroups), dim3(512), 0, st, a1, a2, t1, t2, split,
                     (int)second_first);
}

}  // namespace jf
