// Instantiations of the ring kernel for one operand type, K-contiguous operands.
#include "ring_launch.hpp"

namespace mi355gemm {
#define X(BM, BN, WM, WN, KS, NS, T1, T2) MI355GEMM_RING_DEFINE(f8e4m3_t, bf16_t, BM, BN, WM, WN, KS, NS, true, true)
MI355GEMM_RINGS(X)
#undef X
}  // namespace mi355gemm
