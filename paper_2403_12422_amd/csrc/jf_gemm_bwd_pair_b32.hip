// gemm_pair_kernel instances of block size 32: input gradient and weight gradient of a layer in one launch, numbered as in
// jf_gemm_shapes.hpp (a translation unit of its own for build time).
#include "jf_gemm_fine.hpp"

namespace jf {

template <int WM, int WN>
using Dgrad = GemmInstance<32, WM, WN, 2, 2, true, false>;
template <int WM, int WN>
using Wgrad = GemmInstance<32, WM, WN, 2, 2, false, false>;

void launch_gemm_bwd_pair_b32(const PairChoice& choice, const GemmArgs& dgrad, const GemmArgs& wgrad, hipStream_t st) {
  const int pair = choice.pair;
  if (pair == 21) launch_pair<Dgrad<2, 2>, Wgrad<2, 2>>(dgrad, wgrad, choice, st);
  else if (pair == 22) launch_pair<Dgrad<2, 1>, Wgrad<2, 1>>(dgrad, wgrad, choice, st);
  else if (pair == 26) launch_pair<GemmInstance<32, 1, 1, 4, 2, true, false>, GemmInstance<32, 1, 1, 4, 2, false, false>>(dgrad, wgrad, choice, st);
  else if (pair == 23) launch_pair<Dgrad<1, 1>, Wgrad<1, 1>>(dgrad, wgrad, choice, st);
  else if (pair == 24) launch_pair<FineInstance<true, false>, Wgrad<1, 1>>(dgrad, wgrad, choice, st);
  else launch_pair<Dgrad<1, 1>, FineInstance<false, false>>(dgrad, wgrad, choice, st);
}

}  // namespace jf
