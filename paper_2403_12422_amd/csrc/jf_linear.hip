// Per-block INT8 linear layer (Sec. 5, Alg. 1): C entry points of forward, dgrad, wgrad and the INT32-partial
// test hook.  The kernels live in jf_gemm_kernel.hpp, jf_gemm_fine.hpp and jf_gemm_wide.hpp and are instantiated per product and
// block size in jf_gemm_<product>_b<block>.hip and jf_gemm_bwd_pair_b<block>.hip; jf_gemm_shapes.hpp picks among them.
#include <atomic>

#include "jf_gemm_shapes.hpp"

namespace jf {

static std::atomic<int> g_forced_shape{0};   // test hook, see jf_debug_set_gemm_shape: 0 unless a test sets it

void launch_gemm_fwd_b32(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_fwd_b64(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_fwd_b128(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_dgrad_b32(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_dgrad_b64(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_dgrad_b128(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_wgrad_b32(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_wgrad_b64(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_wgrad_b128(int shape, const GemmArgs& a, bool dump, hipStream_t st);
void launch_gemm_bwd_pair_b32(const PairChoice& choice, const GemmArgs& dgrad, const GemmArgs& wgrad, hipStream_t st);
void launch_gemm_bwd_pair_b64(const PairChoice& choice, const GemmArgs& dgrad, const GemmArgs& wgrad, hipStream_t st);
void launch_gemm_bwd_pair_b128(const PairChoice& choice, const GemmArgs& dgrad, const GemmArgs& wgrad, hipStream_t st);

// Input and weight gradient in one launch, if that is the faster way; false: nothing launched.
static bool launch_bwd_pair(int block, const GemmArgs& dgrad, const GemmArgs& wgrad, hipStream_t st) {
  const PairChoice choice = choose_pair(block, dgrad, wgrad, g_forced_shape.load(std::memory_order_relaxed));
  if (choice.pair == 0) return false;
  if (block == 32) launch_gemm_bwd_pair_b32(choice, dgrad, wgrad, st);
  else if (block == 64) launch_gemm_bwd_pair_b64(choice, dgrad, wgrad, st);
  else launch_gemm_bwd_pair_b128(choice, dgrad, wgrad, st);
  return true;
}

// which: 0 forward, 1 dgrad, 2 wgrad
static void launch_gemm(int which, int block, const GemmArgs& a, bool dump, hipStream_t st) {
  typedef void (*launcher)(int, const GemmArgs&, bool, hipStream_t);
  static const launcher table[3][3] = {
      {launch_gemm_fwd_b32, launch_gemm_fwd_b64, launch_gemm_fwd_b128},
      {launch_gemm_dgrad_b32, launch_gemm_dgrad_b64, launch_gemm_dgrad_b128},
      {launch_gemm_wgrad_b32, launch_gemm_wgrad_b64, launch_gemm_wgrad_b128},
  };
  const int shape = choose_shape(block, (Product)which, a, g_forced_shape.load(std::memory_order_relaxed));
  table[which][block == 32 ? 0 : (block == 64 ? 1 : 2)](shape, a, dump, st);
}

static int32_t check_linear(const void* p0, const void* p1, const void* p2, const void* p3, int64_t N, int64_t C,
                            int64_t D, int32_t block) {
  if (!p0 || !p1 || !p2 || !p3) return JF_ERR_NULL;
  if (!valid_block(block)) return JF_ERR_BLOCK;
  if (!valid_dim(N, block) || !valid_dim(C, block) || !valid_dim(D, block)) return JF_ERR_SHAPE;
  if (!valid_size(N, C) || !valid_size(N, D) || !valid_size(D, C)) return JF_ERR_SHAPE;
  if (!aligned16(p0) || !aligned4(p1) || !aligned16(p2) || !aligned4(p3)) return JF_ERR_ALIGN;
  return JF_OK;
}

static int32_t check_out(const int8_t* q, const float* s, const float* f, bool q_required) {
  if ((q == nullptr) != (s == nullptr)) return JF_ERR_NULL;
  if (q_required && !q) return JF_ERR_NULL;
  if (!q && !f) return JF_ERR_NULL;
  if ((q && !aligned16(q)) || (s && !aligned4(s)) || (f && !aligned16(f))) return JF_ERR_ALIGN;
  return JF_OK;
}

// Operand description of the three products in the canonical out = A Bm^T form.
static GemmArgs make_args(int which, const int8_t* a, const float* sa, const int8_t* b, const float* sb, int64_t N,
                          int64_t C, int64_t D, int32_t block) {
  GemmArgs g{};
  g.A = a; g.SA = sa; g.Bm = b; g.SB = sb;
  if (which == 0) g.M = (int)N, g.Nn = (int)D, g.K = (int)C;        // Y = X W^T: A = X (N x C), Bm = W (D x C), both K-major
  else if (which == 1) g.M = (int)N, g.Nn = (int)C, g.K = (int)D;   // dX = dY W: A = dY (N x D) K-major, Bm = W^T stored as W (D x C)
  else g.M = (int)D, g.Nn = (int)C, g.K = (int)N;                   // dW = dY^T X: A = dY^T stored as dY (N x D), Bm = X^T stored as X (N x C)
  g.set_strides(block, which != 2, which == 0);
  return g;
}

}  // namespace jf

extern "C" int32_t jf_linear_fwd(const int8_t* X, const float* SX, const int8_t* W, const float* SW, int64_t N,
                                 int64_t C, int64_t D, int32_t block, int8_t* Y, float* SY, float* Y_f32, void* ws,
                                 size_t ws_bytes, void* stream) {
  using namespace jf;
  (void)ws; (void)ws_bytes;
  int32_t rc = check_linear(X, SX, W, SW, N, C, D, block);
  if (rc == JF_OK) rc = check_out(Y, SY, Y_f32, true);
  if (rc != JF_OK) return rc;
  GemmArgs g = make_args(0, X, SX, W, SW, N, C, D, block);
  g.Oq = Y; g.Os = SY; g.Of = Y_f32;
  launch_gemm(0, block, g, false, reinterpret_cast<hipStream_t>(stream));
  return launch_status();
}

extern "C" int32_t jf_linear_dgrad(const int8_t* dY, const float* SdY, const int8_t* W, const float* SW, int64_t N,
                                   int64_t C, int64_t D, int32_t block, int8_t* dX, float* SdX, float* dX_f32,
                                   void* ws, size_t ws_bytes, void* stream) {
  using namespace jf;
  (void)ws; (void)ws_bytes;
  int32_t rc = check_linear(dY, SdY, W, SW, N, C, D, block);
  if (rc == JF_OK) rc = check_out(dX, SdX, dX_f32, true);
  if (rc != JF_OK) return rc;
  GemmArgs g = make_args(1, dY, SdY, W, SW, N, C, D, block);
  g.Oq = dX; g.Os = SdX; g.Of = dX_f32;
  launch_gemm(1, block, g, false, reinterpret_cast<hipStream_t>(stream));
  return launch_status();
}

extern "C" int32_t jf_linear_wgrad(const int8_t* dY, const float* SdY, const int8_t* X, const float* SX, int64_t N,
                                   int64_t C, int64_t D, int32_t block, int8_t* dW, float* SdW, float* dW_f32,
                                   void* ws, size_t ws_bytes, void* stream) {
  using namespace jf;
  (void)ws; (void)ws_bytes;
  int32_t rc = check_linear(dY, SdY, X, SX, N, C, D, block);
  if (rc == JF_OK) rc = check_out(dW, SdW, dW_f32, false);
  if (rc != JF_OK) return rc;
  GemmArgs g = make_args(2, dY, SdY, X, SX, N, C, D, block);
  g.Oq = dW; g.Os = SdW; g.Of = dW_f32;
  launch_gemm(2, block, g, false, reinterpret_cast<hipStream_t>(stream));
  return launch_status();
}

extern "C" int32_t jf_linear_bwd(const int8_t* dY, const float* SdY, const int8_t* W, const float* SW, const int8_t* X,
                                 const float* SX, int64_t N, int64_t C, int64_t D, int32_t block, int8_t* dX, float* SdX,
                                 float* dX_f32, int8_t* dW, float* SdW, float* dW_f32, void* ws, size_t ws_bytes,
                                 void* stream) {
  using namespace jf;
  (void)ws; (void)ws_bytes;
  int32_t rc = check_linear(dY, SdY, W, SW, N, C, D, block);
  if (rc == JF_OK) rc = check_linear(dY, SdY, X, SX, N, C, D, block);
  if (rc == JF_OK) rc = check_out(dX, SdX, dX_f32, true);
  if (rc == JF_OK) rc = check_out(dW, SdW, dW_f32, false);
  if (rc != JF_OK) return rc;
  GemmArgs gd = make_args(1, dY, SdY, W, SW, N, C, D, block);
  gd.Oq = dX; gd.Os = SdX; gd.Of = dX_f32;
  GemmArgs gw = make_args(2, dY, SdY, X, SX, N, C, D, block);
  gw.Oq = dW; gw.Os = SdW; gw.Of = dW_f32;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  // dW over W: the input gradient has to have read W before the weight gradient replaces it
  const MemRange weights[] = {{W, D * C}, {SW, D / block * (C / block) * 4}};
  const MemRange grads[] = {{dW, D * C}, {SdW, D / block * (C / block) * 4}, {dW_f32, D * C * 4}};
  if (any_overlap(grads, weights) || !launch_bwd_pair(block, gd, gw, st)) {
    launch_gemm(1, block, gd, false, st);
    rc = launch_status();
    if (rc != JF_OK) return rc;
    launch_gemm(2, block, gw, false, st);
  }
  return launch_status();
}

extern "C" int32_t jf_debug_linear_partials(int32_t which, const int8_t* A, const int8_t* Bm, int64_t N, int64_t C,
                                            int64_t D, int32_t block, int64_t kb, int32_t* out, void* stream) {
  using namespace jf;
  if (!A || !Bm || !out) return JF_ERR_NULL;
  if (which < 0 || which > 2) return JF_ERR_SHAPE;
  if (!valid_block(block)) return JF_ERR_BLOCK;
  if (!valid_dim(N, block) || !valid_dim(C, block) || !valid_dim(D, block)) return JF_ERR_SHAPE;
  if (!valid_size(N, C) || !valid_size(N, D) || !valid_size(D, C)) return JF_ERR_SHAPE;
  if (!aligned16(A) || !aligned16(Bm) || !aligned16(out)) return JF_ERR_ALIGN;
  const int64_t K = which == 0 ? C : (which == 1 ? D : N);
  if (kb < 0 || kb >= K / block) return JF_ERR_SHAPE;
  GemmArgs g = make_args(which, A, nullptr, Bm, nullptr, N, C, D, block);
  g.dump = out;
  g.dump_kb = (int)kb;
  launch_gemm(which, block, g, true, reinterpret_cast<hipStream_t>(stream));
  return launch_status();
}

// A shape or pair that the block size does not have (jf_gemm_shapes.hpp) leaves the choice automatic.
extern "C" int32_t jf_debug_set_gemm_shape(int32_t shape) {
  if (shape != 0 && shape != 1 && shape != 4 && shape != 6 && shape != 7 && shape != 8 && shape != 10 && shape != 11 && (shape < 21 || shape > 26)) return JF_ERR_SHAPE;
  jf::g_forced_shape.store(shape, std::memory_order_relaxed);
  return JF_OK;
}
