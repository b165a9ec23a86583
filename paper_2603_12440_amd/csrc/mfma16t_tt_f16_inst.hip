// Instantiations of the 16x16x32 matrix-core kernel for one operand type and one pair of layouts:
// A column-major, B column-major.
#include "mfma16_launch.hpp"

namespace mi355gemm {
#define X(BM, BN, WM, WN, G, P) MI355GEMM_MFMA16T_DEFINE(f16_t, BM, BN, WM, WN, G, P, false, true)
MI355GEMM_MFMA16T_TILES(X)
#undef X
}  // namespace mi355gemm
