// One-pass LayerNorm kernels of block size 128 (a translation unit of its own for build time).
#include "jf_layernorm_rows.hpp"

JF_LAYERNORM_ROWS_INSTANCE(128)
