// Launcher of the 16x16x32 matrix-core kernel and the list of its compiled tile shapes.  The
// instantiations live in one translation unit per operand type (mfma16_bf16_inst.hip,
// mfma16_f16_inst.hip); the table in gemm_api.hip only refers to them.
#pragma once

#include "plan.hpp"
#include "mfma16_kernel.hpp"

namespace mi355gemm {

// EITHER: the kernel takes both tile orders
template <int BM, int BN, bool EITHER>
MfmaArgs mfma16_args(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias) {
  const gemm_desc_t& d = pl.d;
  MfmaArgs a;
  a.A = A; a.B = B; a.C = C; a.bias = (const float*)bias;
  a.M = (int)d.M; a.N = (int)d.N; a.K = (int)d.K;
  a.lda = d.lda; a.ldb = d.ldb; a.ldc = d.ldc;
  a.stride_a = d.stride_a; a.stride_b = d.stride_b; a.stride_c = d.stride_c;
  a.stride_bias = d.stride_bias;
  a.has_bias = epilogue_has_bias(d.epilogue);
  a.act = epilogue_activation(d.epilogue);
  a.scale = d.scale;
  a.c_f32 = d.dtype_c == GEMM_F32;
  a.c_col = d.layout_c == GEMM_COL_MAJOR;
  a.tiles_m = (int)((d.M + BM - 1) / BM);
  a.tiles_n = (int)((d.N + BN - 1) / BN);
  a.c_cached = pl.c_cached;
  a.batches = (int)d.batch;
  a.touch = touch_shift(a.tiles_n, 4) + (touch_shift(a.tiles_m, 8) << 4);
  set_tile_order<BM, BN, EITHER>(a, pl);
  return a;
}

// A_KF, B_KF: K is the contiguous index of A / B
template <typename T, typename TO, int BM, int BN, int WM, int WN, int G, bool PERSIST, bool A_KF = true, bool B_KF = true, int S = 2>
hipError_t launch_mfma16(const gemm_plan& pl, const void* A, const void* B, void* C,
                         const void* bias, hipStream_t s) {
  const MfmaArgs a = mfma16_args<BM, BN, kEitherOrder<BM, BN, S, PERSIST>>(pl, A, B, C, bias);
  mfma16_gemm_kernel<T, TO, BM, BN, WM, WN, G, PERSIST, A_KF, B_KF, S><<<pl.grid, pl.block, 0, s>>>(a);
  return hipGetLastError();
}

// X(BM, BN, WM, WN, G, PERSIST): tile, wave grid, sub-steps per k-step (slabs of 64 columns of K, two
// stages), one tile per workgroup or a persistent workgroup walking over several
#define MI355GEMM_MFMA16_TILES(X) \
  X(256, 256, 2, 4, 2, false)     \
  X(224, 256, 2, 4, 2, false)     \
  X(192, 256, 2, 4, 2, false)     \
  X(256, 256, 2, 2, 2, false)     \
  X(128, 128, 2, 2, 2, false)
#define MI355GEMM_MFMA16P_TILES(X) \
  X(256, 256, 2, 4, 2, true)       \
  X(224, 256, 2, 4, 2, true)       \
  X(192, 256, 2, 4, 2, true)       \
  X(128, 128, 2, 2, 2, true)
// fp8 operands (slabs of 128 columns, one k-step: four sub-steps)
#define MI355GEMM_MFMA16F8_TILES(X) \
  X(256, 256, 2, 4, 4, false)       \
  X(224, 256, 2, 4, 4, false)       \
  X(192, 256, 2, 4, 4, false)       \
  X(256, 192, 4, 2, 4, false)       \
  X(128, 128, 2, 2, 4, false)
#define MI355GEMM_MFMA16F8P_TILES(X) \
  X(256, 256, 2, 4, 4, true)         \
  X(224, 256, 2, 4, 4, true)         \
  X(192, 256, 2, 4, 4, true)         \
  X(256, 192, 4, 2, 4, true)         \
  X(128, 128, 2, 2, 4, true)

// The same for operands whose K is not contiguous, one translation unit per operand type and layout pair
// (mfma16t_*_inst.hip); the table's entry picks the pair from the plan's layouts.
#define MI355GEMM_MFMA16T_TILES(X) \
  X(256, 256, 2, 4, 2, false)      \
  X(256, 256, 2, 4, 2, true)       \
  X(192, 256, 2, 4, 2, false)      \
  X(192, 256, 2, 4, 2, true)       \
  X(128, 128, 2, 2, 2, false)      \
  X(128, 128, 2, 2, 2, true)
#define MI355GEMM_MFMA16T_DECLARE(T, BM, BN, WM, WN, G, P, AK, BK)                            \
  extern template hipError_t launch_mfma16<T, T, BM, BN, WM, WN, G, P, AK, BK>(                \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);
#define MI355GEMM_MFMA16T_DEFINE(T, BM, BN, WM, WN, G, P, AK, BK)                             \
  template hipError_t launch_mfma16<T, T, BM, BN, WM, WN, G, P, AK, BK>(                       \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

// four slabs in LDS, one workgroup per CU: X(BM, BN, WM, WN, G, S)
#define MI355GEMM_MFMA16S_TILES(X) X(128, 128, 2, 2, 2, 4)
#define MI355GEMM_MFMA16S_DECLARE(T, BM, BN, WM, WN, G, S, AK, BK)                            \
  extern template hipError_t launch_mfma16<T, T, BM, BN, WM, WN, G, false, AK, BK, S>(         \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);
#define MI355GEMM_MFMA16S_DEFINE(T, BM, BN, WM, WN, G, S, AK, BK)                             \
  template hipError_t launch_mfma16<T, T, BM, BN, WM, WN, G, false, AK, BK, S>(                \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

#define MI355GEMM_MFMA16F8S_TILES(X) X(128, 128, 2, 2, 4, 4)
#define MI355GEMM_MFMA16F8S_DECLARE(BM, BN, WM, WN, G, S)                                    \
  extern template hipError_t launch_mfma16<f8e4m3_t, bf16_t, BM, BN, WM, WN, G, false, true, true, S>( \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);
#define MI355GEMM_MFMA16F8S_DEFINE(BM, BN, WM, WN, G, S)                                     \
  template hipError_t launch_mfma16<f8e4m3_t, bf16_t, BM, BN, WM, WN, G, false, true, true, S>( \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

#define MI355GEMM_MFMA16_DECLARE(T, TO, BM, BN, WM, WN, G, P)                               \
  extern template hipError_t launch_mfma16<T, TO, BM, BN, WM, WN, G, P>(                      \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);
#define MI355GEMM_MFMA16_DEFINE(T, TO, BM, BN, WM, WN, G, P)                                \
  template hipError_t launch_mfma16<T, TO, BM, BN, WM, WN, G, P>(                             \
      const gemm_plan&, const void*, const void*, void*, const void*, hipStream_t);

}  // namespace mi355gemm
