// gemm_pair_kernel instances of block size 64: input gradient and weight gradient of a layer in one launch, numbered as in
// jf_gemm_shapes.hpp (a translation unit of its own for build time).
#include "jf_gemm_wide.hpp"

namespace jf {
void launch_gemm_bwd_pair_b64(const PairChoice& choice, const GemmArgs& dgrad, const GemmArgs& wgrad, hipStream_t st) {
  const int pair = choice.pair;
  if (pair == 21) launch_pair<GemmInstance<64, 2, 2, 2, 2, true, false>, GemmInstance<64, 2, 2, 2, 2, false, false>>(dgrad, wgrad, choice, st);
  else if (pair == 26) launch_wide_pair<64>(dgrad, wgrad, st);
  else launch_pair<GemmInstance<64, 1, 1, 2, 2, true, false>, GemmInstance<64, 1, 1, 2, 2, false, false>>(dgrad, wgrad, choice, st);
}
}  // namespace jf
