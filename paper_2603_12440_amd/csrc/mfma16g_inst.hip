// Instantiations of the ring kernel for 16-bit operands of any alignment, every pair of layouts.
#include "ring_launch.hpp"

namespace mi355gemm {
#define X(BM, BN, WM, WN, KS, T1, T2)                    \
  MI355GEMM_MFMA16G_DEFINE(bf16_t, BM, BN, WM, WN, KS)   \
  MI355GEMM_MFMA16G_DEFINE(f16_t, BM, BN, WM, WN, KS)
MI355GEMM_MFMA16G_TILES(X)
#undef X
}  // namespace mi355gemm
