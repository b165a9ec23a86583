// Launcher of the ring kernel and the list of its compiled shapes (instantiated in ring_*_inst.hip).
#pragma once

#include "mfma16_launch.hpp"
#include "ring_kernel.hpp"

namespace mi355gemm {

template <typename T, typename TO, int BM, int BN, int WM, int WN, int KS, int NS, bool A_KF, bool B_KF>
hipError_t launch_ring(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  ring_gemm_kernel<T, TO, BM, BN, WM, WN, KS, NS, A_KF, B_KF><<<pl.grid, pl.block, 0, s>>>(mfma16_args<BM, BN>(pl, A, B, C, bias));
  return hipGetLastError();
}

// X(BM, BN, WM, WN, KS, NSTAGE, t1, t2): t1 and t2 are the microseconds a slab takes (KS * 128 bytes of each row)
// with one workgroup on a CU and with two (0: two do not fit), as measured on 64 x 6144 x 4096 and its neighbours
#define MI355GEMM_RINGS(X)                    \
  X(32, 32, 2, 2, 2, 4, 0.233, 0.34)          \
  X(32, 32, 2, 2, 4, 3, 0.40, 0.0)            \
  X(64, 32, 4, 2, 2, 4, 0.30, 0.0)            \
  MI355GEMM_RINGS_T(X)
// the shapes that also take operands whose K is not contiguous (blocks of 64 rows)
#define MI355GEMM_RINGS_T(X)                  \
  X(64, 64, 2, 4, 2, 4, 0.44, 0.0)            \
  X(64, 64, 2, 4, 1, 5, 0.28, 0.375)
#define MI355GEMM_RING_DECLARE(T, TO, BM, BN, WM, WN, KS, NS, AK, BK)                 \
  extern template hipError_t launch_ring<T, TO, BM, BN, WM, WN, KS, NS, AK, BK>(       \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);
#define MI355GEMM_RING_DEFINE(T, TO, BM, BN, WM, WN, KS, NS, AK, BK)                  \
  template hipError_t launch_ring<T, TO, BM, BN, WM, WN, KS, NS, AK, BK>(              \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

}  // namespace mi355gemm
