// Instantiations of the ring kernel for one operand type, every pair of layouts.
#include "ring_launch.hpp"

namespace mi355gemm {
#define X(BM, BN, WM, WN, KS, NS, T1, T2) MI355GEMM_RING_DEFINE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, true, true)
MI355GEMM_RINGS(X)
MI355GEMM_RINGS16(X)
#undef X
#define X(BM, BN, WM, WN, KS, NS, T1, T2)                                   \
  MI355GEMM_RING_DEFINE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, true, false)  \
  MI355GEMM_RING_DEFINE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, false, false) \
  MI355GEMM_RING_DEFINE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, false, true)
MI355GEMM_RINGS_T(X)
#undef X
#define X(BM, BN, W, NS, T1) MI355GEMM_KSPLIT_INST(, f16_t, BM, BN, W, NS)
MI355GEMM_KSPLITS(X)
#undef X
}  // namespace mi355gemm
