// Instantiations of the 16x16 matrix-core kernel for fp8 operands (a translation unit of its own, so that the operand types
// compile side by side).
#include "mfma16_launch.hpp"

namespace mi355gemm {
#define X(BM, BN, WM, WN, G, P) MI355GEMM_MFMA16_DEFINE(f8e4m3_t, bf16_t, BM, BN, WM, WN, G, P)
MI355GEMM_MFMA16F8_TILES(X)
#undef X
MI355GEMM_MFMA16F8S_TILES(MI355GEMM_MFMA16F8S_DEFINE)
}  // namespace mi355gemm
