// LayerNorm at block size 32 of rows that do not fit a compute unit's registers (more than 2048 columns), still in one pass over
// memory: a workgroup owns 32 whole rows, one workgroup per compute unit, and every wave goes over its strips of 32 x 128 twice, first
// for the row sums, then, last strip first, for the results.  The second time the codes come out of a cache (32 rows of 4096
// columns, forward 128 KB a compute unit: L2; backward 256 KB: the memory-side cache), the last strip's out of registers.
//
// Bound, once memory is read only once, by the vector ALU (backward: 21 instructions per element, up to three waves on a SIMD).
// A wave always has its next strip on the way: as soon as one has moved from LDS to registers, the following one of the order
// below is requested into the same LDS with direct-to-LDS loads, across the passes and across row groups.  As in
// jf_layernorm_rows.hpp a step waits for all its loads and only then stores, so that no wait includes the stores just made.
// Two kernels over strips -> this, in us: forward 8192 x 4096 20.6 -> 16.9, 65536 x 3072 91 -> 77, 131072 x 4096 277 -> 225;
// backward 8192 x 4096 43.8 -> 34.6, 65536 x 3072 223 -> 151.
#include "jf_layernorm_rows.hpp"

namespace jf {

// A wave's place: step s of wave w is strip s waves + w of the row group.  Order of the strips in LDS: 0, 1, ... steps - 1, then
// steps - 2, ... 0, then the next row group's.
struct WideWave {
  int lane, ch, rsub, wave, waves, steps;
  __device__ __forceinline__ WideWave(int strips) {
    lane = threadIdx.x & 63;
    ch = lane & 7;
    rsub = lane >> 3;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    waves = blockDim.x >> 6;
    steps = (strips - wave + waves - 1) / waves;
  }
  __device__ __forceinline__ int c0(int s) const { return (s * waves + wave) * 128; }   // first column of the strip
  __device__ __forceinline__ int col(int s) const { return c0(s) + 16 * ch; }           // of the lane's chunks, inside the matrix or not
};

// LDS of a forward wave: codes, block scales, gamma and beta of the strip in registers and of the one behind it, mean and rstd
constexpr int kWideFwdScale = 4096, kWideFwdGamma = kWideFwdScale + 256, kWideFwdBeta = kWideFwdGamma + 1024, kWideFwdStat = kWideFwdBeta + 1024,
              kWideFwdWaveBytes = kWideFwdStat + 256;

template <StorePolicy SP>
__global__ void __launch_bounds__(1024) layernorm_wide_kernel(const LayerNormRows a) {
  extern __shared__ __align__(16) int8_t smem[];
  const WideWave t(a.strips);
  double* const s_row = reinterpret_cast<double*>(smem);                       // [copy][wave][row][sum]
  int8_t* const own = smem + t.waves * kFwdRowBytes + t.wave * kWideFwdWaveBytes;
  const int groups = a.rows / 32, lc = a.cols / 32;
  int parity = 0;                                      // of the copy of gamma and beta that was requested last
  // results: the strip is for the second pass (too)
  auto request = [&](int g, int s, bool results) __attribute__((always_inline)) {
    const int c0 = t.c0(s), col = t.col(s) < a.cols ? t.col(s) : c0;   // lanes outside the matrix: the strip's first chunk
    const uint32_t off = (uint32_t)(t.rsub * a.cols + col);
    const int8_t* const x = uniform_pointer(a.X + (int64_t)g * 32 * a.cols);
#pragma unroll
    for (int p = 0; p < 4; ++p) load_lds_16(x + (int64_t)p * 8 * a.cols, off, own, 1024 * p);
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SX + (int64_t)g * lc)), (uint32_t)(col / 32) * 4, own, kWideFwdScale);
    if (results) {
      parity ^= 1;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t at = (uint32_t)min(c0 + t.lane + 64 * i, a.cols - 1) * 4;
        load_lds_4(reinterpret_cast<const int8_t*>(a.gamma), at, own, kWideFwdGamma + 512 * parity + 256 * i);
        load_lds_4(reinterpret_cast<const int8_t*>(a.beta), at, own, kWideFwdBeta + 512 * parity + 256 * i);
      }
    }
  };

  request(blockIdx.x, 0, t.steps == 1);
  wait_all_loads();
  int copy = 0;
  for (int g = blockIdx.x; g < groups; g += gridDim.x, copy ^= 1) {
    const int next = g + (int)gridDim.x;
    uint4 px[4];
    float sx;
    int taken;                                         // copy of gamma and beta of the strip in registers
    const auto take = [&](int next_g, int next_s, bool results) __attribute__((always_inline)) {
#pragma unroll
      for (int p = 0; p < 4; ++p) px[p] = *reinterpret_cast<const uint4*>(own + 1024 * p + 16 * t.lane);
      sx = *reinterpret_cast<const float*>(own + kWideFwdScale + 4 * t.lane);
      taken = parity;
      wait_lds();
      if (next_g < groups) request(next_g, next_s, results);
    };
    double s1[4], s2[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) s1[p] = s2[p] = 0.0;
    for (int s = 0; s < t.steps; ++s) {
      if (s + 1 < t.steps) take(g, s + 1, s + 2 == t.steps);
      else take(s == 0 ? next : g, max(s - 1, 0), true);
      const double sd = t.col(s) < a.cols ? (double)sx : 0.0, sd2 = sd * sd;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        int i1, i2;
        chunk_moments(px[p], i1, i2);
        s1[p] = __builtin_fma(sd, (double)i1, s1[p]);
        s2[p] = __builtin_fma(sd2, (double)i2, s2[p]);
      }
      wait_all_loads();
    }
    double* const row = s_row + ((copy * t.waves + t.wave) * 32) * 2;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      s1[p] = wave_group_sum_f64<7>(s1[p]);
      s2[p] = wave_group_sum_f64<7>(s2[p]);
      if (t.ch == 0) *reinterpret_cast<double2*>(row + 2 * (t.rsub + 8 * p)) = make_double2(s1[p], s2[p]);
    }
    lds_barrier();
    {
      const double* v = s_row + ((copy * t.waves) * 32 + (t.lane & 31)) * 2 + (t.lane >> 5);
      const double sum = sum_over_strips(v, t.waves);
      const double other = lane_xor_f64<5>(sum);
      const double mud = (t.lane < 32 ? sum : other) * a.inv_cols;
      const float var = fmaxf((float)((t.lane < 32 ? other : sum) * a.inv_cols - mud * mud), 0.0f);
      const float ve = var + a.eps;
      float rs = __builtin_amdgcn_rsqf(ve);
      rs = rs * __builtin_fmaf(-0.5f * ve * rs, rs, 1.5f);
      if (t.lane < 32) reinterpret_cast<float2*>(own + kWideFwdStat)[t.lane] = make_float2((float)mud, rs);
      wave_lds_fence();
      if (t.wave == 0 && t.lane < 32) {
        a.mean[g * 32 + t.lane] = (float)mud;
        a.rstd[g * 32 + t.lane] = rs;
      }
    }
    for (int s = t.steps - 1; s >= 0; --s) {
      if (s + 1 < t.steps) take(s == 0 ? next : g, max(s - 1, 0), s != 0);
      float k1[4], kb[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float2 st = reinterpret_cast<const float2*>(own + kWideFwdStat)[t.rsub + 8 * p];
        k1[p] = sx * st.y;
        kb[p] = __builtin_fmaf(-128.0f, k1[p], -st.x * st.y);
      }
      float y[4][16];
      float m = 0.0f;
      const float* const gamma = reinterpret_cast<const float*>(own + kWideFwdGamma + 512 * taken) + 16 * t.ch;
      const float* const beta = reinterpret_cast<const float*>(own + kWideFwdBeta + 512 * taken) + 16 * t.ch;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float4 gm = *reinterpret_cast<const float4*>(gamma + 4 * d), bt = *reinterpret_cast<const float4*>(beta + 4 * d);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const uint32_t w = dword_of(px[p], d) ^ 0x80808080u;
          y[p][4 * d + 0] = __builtin_fmaf(__builtin_fmaf((float)(w & 0xffu), k1[p], kb[p]), gm.x, bt.x);
          y[p][4 * d + 1] = __builtin_fmaf(__builtin_fmaf((float)((w >> 8) & 0xffu), k1[p], kb[p]), gm.y, bt.y);
          y[p][4 * d + 2] = __builtin_fmaf(__builtin_fmaf((float)((w >> 16) & 0xffu), k1[p], kb[p]), gm.z, bt.z);
          y[p][4 * d + 3] = __builtin_fmaf(__builtin_fmaf((float)(w >> 24), k1[p], kb[p]), gm.w, bt.w);
        }
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) m = amax16(m, y[p]);
      float scale;
      double inv;
      strip32_block_scale(m, scale, inv);
      uint4 o[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        o[p] = quantize16(y[p], inv);
        asm volatile("" : "+v"(o[p].x), "+v"(o[p].y), "+v"(o[p].z), "+v"(o[p].w));
        __builtin_amdgcn_sched_barrier(0);
      }
      wait_all_loads();
      const int col = t.col(s);
      if (col < a.cols) {
        int8_t* const out = uniform_pointer(a.Y + (int64_t)g * 32 * a.cols);
#pragma unroll
        for (int p = 0; p < 4; ++p)
          store_as_at<SP>(out + (int64_t)p * 8 * a.cols, (uint32_t)(t.rsub * a.cols + col), v4i{(int)o[p].x, (int)o[p].y, (int)o[p].z, (int)o[p].w});
        if ((t.lane & 57) == 0) store_scale<SP>(reinterpret_cast<int8_t*>(uniform_pointer(a.SY + (int64_t)g * lc)) + (col / 32) * 4, scale);
      }
    }
  }
}

// LDS of a backward wave: codes of x and of g, their block scales, mean and rstd of the 32 rows, the two row means, gamma as above,
// and the running column sums of each of its strips
constexpr int kWideG = 4096, kWideScaleX = 8192, kWideScaleG = kWideScaleX + 256, kWideMean = kWideScaleG + 256, kWideRstd = kWideMean + 128,
              kWideMeans = kWideRstd + 128, kWideGamma = kWideMeans + 256, kWideSums = kWideGamma + 1024, kWideStep = 1024;
constexpr int wide_wave_bytes(int steps) { return kWideSums + kWideStep * steps; }

// The column sums of a strip are reduced over the row lanes at once (a wave has too many strips to keep 32 sums a lane for each)
// and added to the wave's own in LDS: 1.5 instructions per element.
template <StorePolicy SP>
__global__ void __launch_bounds__(768) layernorm_bwd_wide_kernel(const LayerNormBwdRows a, int wave_bytes) {
  extern __shared__ __align__(16) int8_t smem[];
  const WideWave t(a.strips);
  float* const s_row = reinterpret_cast<float*>(smem);                         // [copy][wave][row][sum]
  int8_t* const own = smem + t.waves * kBwdRowBytes + t.wave * wave_bytes;
  const int groups = a.rows / 32, lc = a.cols / 32;
  int parity = 0;                                      // of the copy of gamma that was requested last
  auto request = [&](int g, int s) __attribute__((always_inline)) {
    const int col = t.col(s) < a.cols ? t.col(s) : t.c0(s);   // lanes outside the matrix: the strip's first chunk
    const uint32_t off = (uint32_t)(t.rsub * a.cols + col), off_scale = (uint32_t)(col / 32) * 4;
    const int8_t* const x = uniform_pointer(a.X + (int64_t)g * 32 * a.cols);
    const int8_t* const gr = uniform_pointer(a.G + (int64_t)g * 32 * a.cols);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      load_lds_16(x + (int64_t)p * 8 * a.cols, off, own, 1024 * p);
      load_lds_16(gr + (int64_t)p * 8 * a.cols, off, own, kWideG + 1024 * p);
    }
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SX + (int64_t)g * lc)), off_scale, own, kWideScaleX);
    load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.SG + (int64_t)g * lc)), off_scale, own, kWideScaleG);
    parity ^= 1;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      load_lds_4(reinterpret_cast<const int8_t*>(a.gamma), (uint32_t)min(t.c0(s) + t.lane + 64 * i, a.cols - 1) * 4, own,
                 kWideGamma + 512 * parity + 256 * i);
    if (s == 0 && t.lane < 32) {   // 32 floats each
      load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.mean + g * 32)), (uint32_t)t.lane * 4, own, kWideMean);
      load_lds_4(uniform_pointer(reinterpret_cast<const int8_t*>(a.rstd + g * 32)), (uint32_t)t.lane * 4, own, kWideRstd);
    }
  };

  request(blockIdx.x, 0);
  float* const sums = reinterpret_cast<float*>(own + kWideSums);
  for (int i = t.lane; i < t.steps * 256; i += 64) sums[i] = 0.0f;
  wait_all_loads();
  wave_lds_fence();

  const int place = reduced_column(t.lane);
  int copy = 0;
  for (int g = blockIdx.x; g < groups; g += gridDim.x, copy ^= 1) {
    uint4 px[4], pg[4];
    float sx, sg, mu[4], rs[4];
    const float* gamma;
    // a strip from LDS to registers, and the request of the one after it
    const auto take = [&](int s, int next_g, int next_s) __attribute__((always_inline)) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        px[p] = *reinterpret_cast<const uint4*>(own + 1024 * p + 16 * t.lane);
        pg[p] = *reinterpret_cast<const uint4*>(own + kWideG + 1024 * p + 16 * t.lane);
      }
      sx = *reinterpret_cast<const float*>(own + kWideScaleX + 4 * t.lane);
      sg = *reinterpret_cast<const float*>(own + kWideScaleG + 4 * t.lane);
      gamma = reinterpret_cast<const float*>(own + kWideGamma + 512 * parity);
      wait_lds();
      if (next_g < groups) request(next_g, next_s);
      sg = t.col(s) < a.cols ? sg : 0.0f;   // what lies outside adds nothing to the sums
    };
    const int next = g + (int)gridDim.x;
    float m1[4], m2[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) m1[p] = m2[p] = 0.0f;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      mu[p] = reinterpret_cast<const float*>(own + kWideMean)[t.rsub + 8 * p];
      rs[p] = reinterpret_cast<const float*>(own + kWideRstd)[t.rsub + 8 * p];
    }
    for (int s = 0; s < t.steps; ++s) {
      const bool last = s + 1 == t.steps;
      take(s, last && s == 0 ? next : g, last ? max(s - 1, 0) : s + 1);
      float cgs[16], cbs[16], kx[4], cx[4], n1[4], n2[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        kx[p] = sx * rs[p];
        cx[p] = -mu[p] * rs[p];
        n1[p] = n2[p] = 0.0f;
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float4 gm4 = *reinterpret_cast<const float4*>(gamma + 16 * t.ch + 4 * d);
        const float gm[4] = {gm4.x, gm4.y, gm4.z, gm4.w};
        float tg[4], tb[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          float x[4], gr[4];
          unpack4(dword_of(px[p], d), x);
          unpack4(dword_of(pg[p], d), gr);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float xh = __builtin_fmaf(x[e], kx[p], cx[p]), gh = gr[e] * gm[e];
            asm volatile("v_add_f32 %0, %0, %1" : "+v"(n1[p]) : "v"(gh));
            asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(n2[p]) : "v"(gh), "v"(xh));
            tg[e] = p == 0 ? gr[e] * xh : __builtin_fmaf(gr[e], xh, tg[e]);
            if (p == 0) tb[e] = gr[e];
            else asm volatile("v_add_f32 %0, %0, %1" : "+v"(tb[e]) : "v"(gr[e]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          cgs[4 * d + e] = sg * tg[e];
          cbs[4 * d + e] = sg * tb[e];
        }
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        m1[p] = __builtin_fmaf(n1[p], sg, m1[p]);
        m2[p] = __builtin_fmaf(n2[p], sg, m2[p]);
      }
      float part[8];
      reduce_rows32(cgs, cbs, part);
      if ((t.lane & 8) == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sums[256 * s + 128 * (j / 4) + j % 4 + place] += part[j];
      }
      wait_all_loads();
    }
    float* const row = s_row + ((copy * t.waves + t.wave) * 32) * 2;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      m1[p] = wave_group_sum<7>(m1[p]);
      m2[p] = wave_group_sum<7>(m2[p]);
      if (t.ch == 0) *reinterpret_cast<float2*>(row + 2 * (t.rsub + 8 * p)) = make_float2(m1[p], m2[p]);
    }
    lds_barrier();
    {
      const float* v = s_row + ((copy * t.waves) * 32 + (t.lane & 31)) * 2 + (t.lane >> 5);
      reinterpret_cast<float*>(own + kWideMeans)[2 * (t.lane & 31) + (t.lane >> 5)] = sum_over_strips(v, t.waves) * a.inv_cols;
      wave_lds_fence();
    }
    float q1[4], q2[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float2 q = reinterpret_cast<const float2*>(own + kWideMeans)[t.rsub + 8 * p];
      q1[p] = q.x;
      q2[p] = q.y;
    }
    for (int s = t.steps - 1; s >= 0; --s) {
      if (s + 1 < t.steps) take(s, s == 0 ? next : g, max(s - 1, 0));   // the last strip is still in registers
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        asm volatile("" : "+v"(px[p].x), "+v"(px[p].y), "+v"(px[p].z), "+v"(px[p].w));
        asm volatile("" : "+v"(pg[p].x), "+v"(pg[p].y), "+v"(pg[p].z), "+v"(pg[p].w));
      }
      float y[4][16], kxm[4], krow[4], rsg[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float kx = sx * rs[p], cx = -mu[p] * rs[p];
        kxm[p] = -rs[p] * q2[p] * kx;
        krow[p] = -rs[p] * __builtin_fmaf(cx, q2[p], q1[p]);
        rsg[p] = rs[p] * sg;
      }
      float m = 0.0f;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float4 gm4 = *reinterpret_cast<const float4*>(gamma + 16 * t.ch + 4 * d);
        const float gm[4] = {gm4.x, gm4.y, gm4.z, gm4.w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          float x[4], gr[4];
          unpack4(dword_of(px[p], d), x);
          unpack4(dword_of(pg[p], d), gr);
#pragma unroll
          for (int e = 0; e < 4; ++e) y[p][4 * d + e] = __builtin_fmaf(x[e], kxm[p], __builtin_fmaf(gr[e] * gm[e], rsg[p], krow[p]));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) m = amax16(m, y[p]);
      float scale;
      double inv;
      strip32_block_scale(m, scale, inv);
      uint4 o[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        o[p] = quantize16(y[p], inv);
        asm volatile("" : "+v"(o[p].x), "+v"(o[p].y), "+v"(o[p].z), "+v"(o[p].w));
        __builtin_amdgcn_sched_barrier(0);
      }
      wait_all_loads();
      const int col = t.col(s);
      if (col < a.cols) {
        const uint32_t off = (uint32_t)(t.rsub * a.cols + col);
        int8_t* const out = uniform_pointer(a.dX + (int64_t)g * 32 * a.cols);
#pragma unroll
        for (int p = 0; p < 4; ++p) store_as_at<SP>(out + (int64_t)p * 8 * a.cols, off, v4i{(int)o[p].x, (int)o[p].y, (int)o[p].z, (int)o[p].w});
        if ((t.lane & 57) == 0) store_scale<SP>(reinterpret_cast<int8_t*>(uniform_pointer(a.SdX + (int64_t)g * lc)) + (col / 32) * 4, scale);
      }
    }
  }
  wave_lds_fence();
  for (int s = 0; s < t.steps; ++s) {
    float* dst = a.partials + (int64_t)blockIdx.x * 2 * a.cols;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = t.c0(s) + t.lane + 64 * (i & 1);
      if (c < a.cols) dst[(i >> 1) * a.cols + c] = sums[256 * s + 64 * i + t.lane];
    }
  }
}

// ------------------------------------------------------------------------------------------------ host
// see launch_rows
template <auto KERNEL, class... Args>
static void launch_wide(int grid, int waves, int bytes, hipStream_t st, const Args&... args) {
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return;
  hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(64 * waves), bytes, st, args...);
}

// Waves: as many as LDS holds with the sums of all their strips, at most twelve (for the registers).
int launch_layernorm_bwd_wide(LayerNormBwdRows a, hipStream_t st) {
  a.strips = (a.cols + 127) / 128;
  a.inv_cols = 1.0f / (float)a.cols;
  const auto waves = [&](int steps) { return (a.strips + steps - 1) / steps; };
  const auto bytes = [&](int steps) { return waves(steps) * (kBwdRowBytes + wide_wave_bytes(steps)); };
  int steps = 2;
  while (waves(steps) > 12 || bytes(steps) > 160 * 1024) ++steps;   // (ends: kLayerNormWideCols)
  static_assert(6 * (kBwdRowBytes + wide_wave_bytes((kLayerNormWideCols / 128 + 5) / 6)) <= 160 * 1024, "six waves share the longest rows");
  const int grid = std::min(a.rows / 32, 256);
  with_store_policy(a.rows, a.cols, [&](auto sp) {
    launch_wide<layernorm_bwd_wide_kernel<decltype(sp)::value>>(grid, waves(steps), bytes(steps), st, a, wide_wave_bytes(steps));
  });
  return grid;
}

void launch_layernorm_wide(LayerNormRows a, hipStream_t st) {
  a.strips = (a.cols + 127) / 128;
  a.inv_cols = 1.0 / (double)a.cols;
  const int steps = (a.strips + 15) / 16, waves = (a.strips + steps - 1) / steps;
  with_store_policy(a.rows, a.cols, [&](auto sp) {
    launch_wide<layernorm_wide_kernel<decltype(sp)::value>>(std::min(a.rows / 32, 256), waves, waves * (kFwdRowBytes + kWideFwdWaveBytes), st, a);
  });
}

}  // namespace jf
