// gemm_kernel instances of the dgrad product at block size 32 (a translation unit of its own for build time).
#include "jf_gemm_fine.hpp"

JF_GEMM_INSTANCE(launch_gemm_dgrad_b32, 32, true, false)
