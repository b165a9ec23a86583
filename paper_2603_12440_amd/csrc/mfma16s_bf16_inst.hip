// Instantiations of the 16x16x32 matrix-core kernel with more than two slabs in LDS, every pair of layouts.
#include "mfma16_launch.hpp"

namespace mi355gemm {
#define X(BM, BN, WM, WN, G, S)                                        \
  MI355GEMM_MFMA16S_DEFINE(bf16_t, BM, BN, WM, WN, G, S, true, true)   \
  MI355GEMM_MFMA16S_DEFINE(bf16_t, BM, BN, WM, WN, G, S, true, false)  \
  MI355GEMM_MFMA16S_DEFINE(bf16_t, BM, BN, WM, WN, G, S, false, false) \
  MI355GEMM_MFMA16S_DEFINE(bf16_t, BM, BN, WM, WN, G, S, false, true)
MI355GEMM_MFMA16S_TILES(X)
#undef X
}  // namespace mi355gemm
