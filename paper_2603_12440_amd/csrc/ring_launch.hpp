// Launcher of the ring kernel and the list of its compiled shapes (instantiated in ring_*_inst.hip).
#pragma once

#include "ksplit_ring_kernel.hpp"
#include "mfma16_launch.hpp"

namespace mi355gemm {

template <typename T, typename TO, int BM, int BN, int WM, int WN, int KS, int NS, bool A_KF, bool B_KF>
hipError_t launch_ring(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  ring_gemm_kernel<T, TO, BM, BN, WM, WN, KS, NS, A_KF, B_KF><<<pl.grid, pl.block, 0, s>>>(mfma16_args<BM, BN, kEitherOrder<BM, BN, NS, false>>(pl, A, B, C, bias));
  return hipGetLastError();
}

// waves that split K (instantiated in ring_*_inst.hip): X(BM, BN, WAVES, NSTAGE, t1), t1 as below
template <typename T, int BM, int BN, int WAVES, int NS>
hipError_t launch_ksplit(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  ksplit_ring_kernel<T, BM, BN, WAVES, NS><<<pl.grid, pl.block, 0, s>>>(mfma16_args<BM, BN, false>(pl, A, B, C, bias));
  return hipGetLastError();
}
#define MI355GEMM_KSPLITS(X) \
  X(64, 64, 8, 1, 0.235)     \
  X(32, 32, 4, 4, 0.088)
#define MI355GEMM_KSPLIT_INST(EXTERN, T, BM, BN, W, NS) \
  EXTERN template hipError_t launch_ksplit<T, BM, BN, W, NS>(const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

// X(BM, BN, WM, WN, KS, NSTAGE, t1, t2): t1 and t2 are the microseconds a slab takes (KS * 128 bytes of each row)
// with one workgroup on a CU and with two (0: two do not fit), as measured on 64 x 6144 x 4096 and its neighbours
#define MI355GEMM_RINGS(X)                    \
  X(32, 32, 2, 2, 2, 4, 0.233, 0.34)          \
  X(32, 32, 2, 2, 4, 3, 0.40, 0.0)            \
  X(64, 32, 4, 2, 2, 4, 0.30, 0.0)            \
  MI355GEMM_RINGS_T(X)
// 16-bit operands only: a barrier per 256 values of K instead of 128.  64x6144x4096 12.5 -> 11.9 us with operands in the last-level
// cache, 16.8 -> 16.6 from HBM; 128x4096x4096 12.6 -> 11.8 and 16.2 -> 15.8.  Six slabs of 128 values were slower (13.5, 17.3).
#define MI355GEMM_RINGS16(X) X(64, 32, 4, 2, 4, 3, 0.565, 0.0)
// the shapes that also take operands whose K is not contiguous (blocks of 64 rows)
#define MI355GEMM_RINGS_T(X)                  \
  X(64, 64, 2, 4, 2, 4, 0.44, 0.0)            \
  X(64, 64, 2, 4, 1, 5, 0.28, 0.375)
// operands of any alignment: X(BM, BN, WM, WN, KS, t1, t2)
template <typename T, int BM, int BN, int WM, int WN, int KS>
hipError_t launch_mfma16g(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  const MfmaArgs a = mfma16_args<BM, BN, kEitherOrder<BM, BN, 2, false>>(pl, A, B, C, bias);
  const bool ak = pl.d.layout_a == GEMM_ROW_MAJOR, bk = pl.d.layout_b == GEMM_COL_MAJOR;
  if (ak && bk) ring_gemm_kernel<T, T, BM, BN, WM, WN, KS, 2, true, true, false><<<pl.grid, pl.block, 0, s>>>(a);
  else if (ak) ring_gemm_kernel<T, T, BM, BN, WM, WN, KS, 2, true, false, false><<<pl.grid, pl.block, 0, s>>>(a);
  else if (bk) ring_gemm_kernel<T, T, BM, BN, WM, WN, KS, 2, false, true, false><<<pl.grid, pl.block, 0, s>>>(a);
  else ring_gemm_kernel<T, T, BM, BN, WM, WN, KS, 2, false, false, false><<<pl.grid, pl.block, 0, s>>>(a);
  return hipGetLastError();
}
#define MI355GEMM_MFMA16G_TILES(X)     \
  X(64, 64, 2, 2, 1, 0.40, 0.50)       \
  X(128, 128, 2, 4, 1, 0.80, 1.0)
#define MI355GEMM_MFMA16G_DECLARE(T, BM, BN, WM, WN, KS)                               \
  extern template hipError_t launch_mfma16g<T, BM, BN, WM, WN, KS>(                    \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);
#define MI355GEMM_MFMA16G_DEFINE(T, BM, BN, WM, WN, KS)                                \
  template hipError_t launch_mfma16g<T, BM, BN, WM, WN, KS>(                           \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

#define MI355GEMM_RING_DECLARE(T, TO, BM, BN, WM, WN, KS, NS, AK, BK)                 \
  extern template hipError_t launch_ring<T, TO, BM, BN, WM, WN, KS, NS, AK, BK>(       \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);
#define MI355GEMM_RING_DEFINE(T, TO, BM, BN, WM, WN, KS, NS, AK, BK)                  \
  template hipError_t launch_ring<T, TO, BM, BN, WM, WN, KS, NS, AK, BK>(              \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

}  // namespace mi355gemm
