// Micro-benchmark of the GEMM's inner pattern with true data dependences and no memory traffic: two INT32 tiles in
// ordinary VGPRs (as in the GEMM kernel) rotate; per unit a chain of B/32 MFMAs runs into one tile while the other,
// which the previous chain wrote, is folded (16 cvt + 16 fmac, Sec. 5.3), a share of the fold after every MFMA.
// The rates it prints are the ceilings the GEMM's K loop is compared with: with operands of a few small numbers, alike in all lanes, and with
// random codes as of a quantized Gaussian tensor, four fragments of each operand in turn, which toggle more bits and so draw more power: under
// the power limit the clock falls, and the same instructions take longer.
// Two orders of the fold: in groups of four conversions and their FMAs, a share after every MFMA; and by halves, all conversions and then all FMAs after
// the last MFMA of the chain, a wave in its FMAs before one in its conversions (s_setprio), as the products on 256x256 tiles at block 64 have it.
#include <hip/hip_runtime.h>
#include <cstdio>
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

__device__ int codes(unsigned n) {   // four codes, each the sum of four random numbers -32 .. 31
  unsigned packed = 0;
  for (int i = 0; i < 4; ++i) {
    unsigned h = (4 * n + i) * 2654435761u + 12345u;
    h ^= h >> 15, h *= 2246822519u, h ^= h >> 13, h *= 3266489917u, h ^= h >> 16;
    const int sum = (int)(h & 63) + (int)(h >> 6 & 63) + (int)(h >> 12 & 63) + (int)(h >> 18 & 63) - 126;
    packed |= (unsigned)(sum & 255) << 8 * i;
  }
  return (int)packed;
}

template <int NC, bool RANDOM, bool HALVES>
__global__ void __launch_bounds__(256) k(int iters, int* out, int seed) {
  constexpr int SETS = RANDOM ? 4 : 1;
  v4i as[SETS], bs[SETS];
  for (int j = 0; j < SETS; ++j) {
    as[j] = v4i{seed + (int)threadIdx.x, seed * 3, seed * 5, seed * 7}, bs[j] = v4i{seed * 11, seed * 13, (int)threadIdx.x, seed};
    if (RANDOM)
      for (int d = 0; d < 4; ++d) {
        as[j][d] = codes(8 * (blockIdx.x * 1024 + threadIdx.x * 4 + j) + d);
        bs[j][d] = codes(8 * (blockIdx.x * 1024 + threadIdx.x * 4 + j) + 4 + d);
      }
  }
  v16i T0 = {0}, T1 = {0};
  float acc[16];
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float t = 1.0f + seed;
#define MFMA0(dst, J) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, 0" : "=v"(dst) : "v"(as[(J) % SETS]), "v"(bs[(J) % SETS]))
#define MFMAC(dst, J) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(dst) : "v"(as[(J) % SETS]), "v"(bs[(J) % SETS]))
#define FOLD(src, R0, R1)                                                                      \
  _Pragma("unroll") for (int r = R0; r < R1; ++r) {                                            \
    float c;                                                                                   \
    asm volatile("v_cvt_f32_i32 %0, %1" : "=v"(c) : "v"(src[r]));                              \
    asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(acc[r]) : "v"(t), "v"(c));                     \
  }
#define BY_HALVES(src)                                                                                                          \
  {                                                                                                                              \
    float c[16];                                                                                                                 \
    __builtin_amdgcn_s_setprio(0);                                                                                               \
    _Pragma("unroll") for (int r = 0; r < 16; ++r) asm volatile("v_cvt_f32_i32 %0, %1" : "=v"(c[r]) : "v"(src[r]));              \
    __builtin_amdgcn_s_setprio(1);                                                                                               \
    _Pragma("unroll") for (int r = 0; r < 16; ++r) asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(acc[r]) : "v"(t), "v"(c[r]));      \
  }
#define CHAIN(dst, J) MFMA0(dst, J); _Pragma("unroll") for (int j = 1; j < NC; ++j) MFMAC(dst, (J) + j);
  for (int it = 0; it < iters; ++it) {
    if (HALVES) {
      CHAIN(T0, 0) BY_HALVES(T1) CHAIN(T1, NC) BY_HALVES(T0) CHAIN(T0, 2 * NC) BY_HALVES(T1) CHAIN(T1, 3 * NC) BY_HALVES(T0)
    } else if (NC == 1) {
      MFMA0(T0, 0); FOLD(T1, 0, 16)
      MFMA0(T1, 1); FOLD(T0, 0, 16)
      MFMA0(T0, 2); FOLD(T1, 0, 16)
      MFMA0(T1, 3); FOLD(T0, 0, 16)
    } else if (NC == 2) {
      MFMA0(T0, 0); FOLD(T1, 0, 8) MFMAC(T0, 1); FOLD(T1, 8, 16)
      MFMA0(T1, 2); FOLD(T0, 0, 8) MFMAC(T1, 3); FOLD(T0, 8, 16)
      MFMA0(T0, 0); FOLD(T1, 0, 8) MFMAC(T0, 1); FOLD(T1, 8, 16)
      MFMA0(T1, 2); FOLD(T0, 0, 8) MFMAC(T1, 3); FOLD(T0, 8, 16)
    } else {
      MFMA0(T0, 0); FOLD(T1, 0, 4) MFMAC(T0, 1); FOLD(T1, 4, 8) MFMAC(T0, 2); FOLD(T1, 8, 12) MFMAC(T0, 3); FOLD(T1, 12, 16)
      MFMA0(T1, 0); FOLD(T0, 0, 4) MFMAC(T1, 1); FOLD(T0, 4, 8) MFMAC(T1, 2); FOLD(T0, 8, 12) MFMAC(T1, 3); FOLD(T0, 12, 16)
      MFMA0(T0, 0); FOLD(T1, 0, 4) MFMAC(T0, 1); FOLD(T1, 4, 8) MFMAC(T0, 2); FOLD(T1, 8, 12) MFMAC(T0, 3); FOLD(T1, 12, 16)
      MFMA0(T1, 0); FOLD(T0, 0, 4) MFMAC(T1, 1); FOLD(T0, 4, 8) MFMAC(T1, 2); FOLD(T0, 8, 12) MFMAC(T1, 3); FOLD(T0, 12, 16)
    }
  }
  float s = 0;
  for (int r = 0; r < 16; ++r) s += acc[r] + T0[r] + T1[r];
  if (s == 1.2345f) out[0] = (int)s;
}

template <int NC, bool RANDOM, bool HALVES = false>
void run(int wps) {
  int* out; (void)hipMalloc(&out, 4);
  const int iters = 40000;   // 10 ms and more, in front of it as long: the clock has come to rest
  hipEvent_t e0, e1; (void)hipEventCreate(&e0); (void)hipEventCreate(&e1);
  k<NC, RANDOM, HALVES><<<256 * wps, 256>>>(iters, out, 1);
  (void)hipDeviceSynchronize();
  (void)hipEventRecord(e0);
  k<NC, RANDOM, HALVES><<<256 * wps, 256>>>(iters, out, 1);
  (void)hipEventRecord(e1);
  (void)hipDeviceSynchronize();
  float ms; (void)hipEventElapsedTime(&ms, e0, e1);
  double ns = ms * 1e6 / iters / wps / (4 * NC);
  printf("block %3d (chain of %d), tiles in VGPRs, %s%s%d waves/SIMD: %6.1f ns per MFMA -> %6.0f TOP/s\n", 32 * NC, NC, RANDOM ? "random codes, " : "",
         HALVES ? "by halves, " : "", wps, ns,
         65536.0 * 1024 / (ns * 1e-9) * 1e-12);
  (void)hipFree(out);
}

int main() {
  for (int w : {2, 3, 4}) { run<1, false>(w); run<2, false>(w); run<4, false>(w); }
  for (int w : {2, 3, 4}) { run<1, true>(w); run<2, true>(w); run<4, true>(w); }
  for (int w : {2, 3, 4}) { run<1, false, true>(w); run<2, false, true>(w); run<4, false, true>(w); }
  for (int w : {2, 3, 4}) { run<1, true, true>(w); run<2, true, true>(w); run<4, true, true>(w); }
  return 0;
}
