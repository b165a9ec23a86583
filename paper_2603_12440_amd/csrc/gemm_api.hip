// Host side of the mi355gemm C ABI (include/gemm.h): descriptor validation, the
// table of compiled kernel instantiations, the choice among them, and launches.
//
// The table-plus-dispatcher shape follows the paper's templated kernels
// (Sec. 3.4 and the templated-kernel example in the appendix): every tile
// shape is a template instantiation, a dispatch function maps integer
// parameters to the instantiation, and a tuner may time each applicable one.
#include <hip/hip_runtime.h>

#include <atomic>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/gemm.h"
#include "common.hpp"
#include "plan.hpp"
#include "mfma_launch.hpp"
#include "mfma16_launch.hpp"
#include "simt_kernel.hpp"
#include "general_mfma_kernel.hpp"
#include "f32_mfma_kernel.hpp"
#include "f32_ring_kernel.hpp"
#include "skinny_kernel.hpp"
#include "ring_launch.hpp"
#include "splitk_kernel.hpp"
#include "device_check.hpp"

using namespace mi355gemm;

namespace mi355gemm {
#define X(BM, BN, BK, WM, WN, NS) MI355GEMM_MFMA_DECLARE(bf16_t, bf16_t, BM, BN, BK, WM, WN, NS) \
                                 MI355GEMM_MFMA_DECLARE(f16_t, f16_t, BM, BN, BK, WM, WN, NS)
MI355GEMM_MFMA_TILES(X)
#undef X
#define X(BM, BN, WM, WN, G, P) MI355GEMM_MFMA16_DECLARE(f8e4m3_t, bf16_t, BM, BN, WM, WN, G, P)
MI355GEMM_MFMA16F8_TILES(X)
MI355GEMM_MFMA16F8P_TILES(X)
#undef X
MI355GEMM_MFMA16F8S_TILES(MI355GEMM_MFMA16F8S_DECLARE)
#define X(BM, BN, WM, WN, G, P) MI355GEMM_MFMA16_DECLARE(bf16_t, bf16_t, BM, BN, WM, WN, G, P) \
                                MI355GEMM_MFMA16_DECLARE(f16_t, f16_t, BM, BN, WM, WN, G, P)
MI355GEMM_MFMA16_TILES(X)
MI355GEMM_MFMA16P_TILES(X)
#undef X
#define X(BM, BN, WM, WN, G, P)                                        \
  MI355GEMM_MFMA16T_DECLARE(bf16_t, BM, BN, WM, WN, G, P, true, false)  \
  MI355GEMM_MFMA16T_DECLARE(bf16_t, BM, BN, WM, WN, G, P, false, false) \
  MI355GEMM_MFMA16T_DECLARE(bf16_t, BM, BN, WM, WN, G, P, false, true)  \
  MI355GEMM_MFMA16T_DECLARE(f16_t, BM, BN, WM, WN, G, P, true, false)   \
  MI355GEMM_MFMA16T_DECLARE(f16_t, BM, BN, WM, WN, G, P, false, false)  \
  MI355GEMM_MFMA16T_DECLARE(f16_t, BM, BN, WM, WN, G, P, false, true)
MI355GEMM_MFMA16T_TILES(X)
#undef X
#define X(BM, BN, WM, WN, KS, NS, T1, T2)                                    \
  MI355GEMM_RING_DECLARE(bf16_t, bf16_t, BM, BN, WM, WN, KS, NS, true, true) \
  MI355GEMM_RING_DECLARE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, true, true)   \
  MI355GEMM_RING_DECLARE(f8e4m3_t, bf16_t, BM, BN, WM, WN, KS, NS, true, true)
MI355GEMM_RINGS(X)
#undef X
#define X(BM, BN, WM, WN, KS, NS, T1, T2)                                    \
  MI355GEMM_RING_DECLARE(bf16_t, bf16_t, BM, BN, WM, WN, KS, NS, true, true) \
  MI355GEMM_RING_DECLARE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, true, true)
MI355GEMM_RINGS16(X)
#undef X
#define X(BM, BN, W, NS, T1)                              \
  MI355GEMM_KSPLIT_INST(extern, bf16_t, BM, BN, W, NS)    \
  MI355GEMM_KSPLIT_INST(extern, f16_t, BM, BN, W, NS)
MI355GEMM_KSPLITS(X)
#undef X
#define X(BM, BN, WM, WN, KS, NS, T1, T2)                                      \
  MI355GEMM_RING_DECLARE(bf16_t, bf16_t, BM, BN, WM, WN, KS, NS, true, false)  \
  MI355GEMM_RING_DECLARE(bf16_t, bf16_t, BM, BN, WM, WN, KS, NS, false, false) \
  MI355GEMM_RING_DECLARE(bf16_t, bf16_t, BM, BN, WM, WN, KS, NS, false, true)  \
  MI355GEMM_RING_DECLARE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, true, false)    \
  MI355GEMM_RING_DECLARE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, false, false)   \
  MI355GEMM_RING_DECLARE(f16_t, f16_t, BM, BN, WM, WN, KS, NS, false, true)
MI355GEMM_RINGS_T(X)
#undef X
#define X(BM, BN, WM, WN, KS, T1, T2)                    \
  MI355GEMM_MFMA16G_DECLARE(bf16_t, BM, BN, WM, WN, KS)  \
  MI355GEMM_MFMA16G_DECLARE(f16_t, BM, BN, WM, WN, KS)
MI355GEMM_MFMA16G_TILES(X)
#undef X
#define X(BM, BN, WM, WN, G, S)                                         \
  MI355GEMM_MFMA16S_DECLARE(bf16_t, BM, BN, WM, WN, G, S, true, true)   \
  MI355GEMM_MFMA16S_DECLARE(bf16_t, BM, BN, WM, WN, G, S, true, false)  \
  MI355GEMM_MFMA16S_DECLARE(bf16_t, BM, BN, WM, WN, G, S, false, false) \
  MI355GEMM_MFMA16S_DECLARE(bf16_t, BM, BN, WM, WN, G, S, false, true)  \
  MI355GEMM_MFMA16S_DECLARE(f16_t, BM, BN, WM, WN, G, S, true, true)    \
  MI355GEMM_MFMA16S_DECLARE(f16_t, BM, BN, WM, WN, G, S, true, false)   \
  MI355GEMM_MFMA16S_DECLARE(f16_t, BM, BN, WM, WN, G, S, false, false)  \
  MI355GEMM_MFMA16S_DECLARE(f16_t, BM, BN, WM, WN, G, S, false, true)
MI355GEMM_MFMA16S_TILES(X)
#undef X
}  // namespace mi355gemm

namespace {

int num_cus();

// ---- launchers ---------------------------------------------------------------------

// the argument block of the general kernels: layouts become element strides
SimtArgs simt_args(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias) {
  const gemm_desc_t& d = pl.d;
  SimtArgs a;
  a.A = A; a.B = B; a.C = C; a.bias = (const float*)bias;
  a.M = d.M; a.N = d.N; a.K = d.K;
  a.a_si = d.layout_a == GEMM_ROW_MAJOR ? d.lda : 1;
  a.a_sk = d.layout_a == GEMM_ROW_MAJOR ? 1 : d.lda;
  a.b_sk = d.layout_b == GEMM_ROW_MAJOR ? d.ldb : 1;
  a.b_sj = d.layout_b == GEMM_ROW_MAJOR ? 1 : d.ldb;
  a.c_si = d.layout_c == GEMM_ROW_MAJOR ? d.ldc : 1;
  a.c_sj = d.layout_c == GEMM_ROW_MAJOR ? 1 : d.ldc;
  a.stride_a = d.stride_a; a.stride_b = d.stride_b; a.stride_c = d.stride_c;
  a.stride_bias = d.stride_bias;
  a.has_bias = epilogue_has_bias(d.epilogue);
  a.act = epilogue_activation(d.epilogue);
  a.scale = d.scale;
  return a;
}

template <typename TIn, typename TOut, int TM, int TN, int TK>
hipError_t launch_simt_typed(const gemm_plan& pl, const void* A, const void* B, void* C,
                             const void* bias, hipStream_t s) {
  const SimtArgs a = simt_args(pl, A, B, C, bias);
  simt_gemm_kernel<TIn, TOut, TM, TN, TK><<<pl.grid, pl.block, 0, s>>>(a);
  return hipGetLastError();
}

template <typename TIn, typename TOut, int TM, int TN, int TK>
hipError_t launch_general_mfma_typed(const gemm_plan& pl, const void* A, const void* B, void* C,
                                     const void* bias, hipStream_t s) {
  const SimtArgs a = simt_args(pl, A, B, C, bias);
  general_mfma_kernel<TIn, TOut, TM, TN, TK><<<pl.grid, pl.block, 0, s>>>(a);
  return hipGetLastError();
}

// Does an fp32 problem on the general kernels' grid run on f32_any_kernel?  (Offsets inside a slab have to fit 32 bits.)
bool f32_takes_any(const gemm_desc_t& d, int tile) {
  const int64_t lim = (int64_t)1 << 32, kMax = ((int64_t)1 << 31) - 512;
  return d.dtype_a == GEMM_F32 && (tile + 1) * d.lda * 4 < lim && (tile + 1) * d.ldb * 4 < lim && d.M < kMax && d.N < kMax && d.K < kMax;
}

template <int TM>
hipError_t launch_f32_any(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  const gemm_desc_t& d = pl.d;
  const SimtArgs a = simt_args(pl, A, B, C, bias);
  MfmaArgs r = mfma16_args<TM, TM, false>(pl, A, B, C, bias);
  r.xcd_remap = d.batch == 1 || (r.tiles_m * (int64_t)r.tiles_n) % 8 == 0;
  const bool ak = d.layout_a == GEMM_ROW_MAJOR, bk = d.layout_b == GEMM_COL_MAJOR;   // K contiguous?
  constexpr int MT = TM / 64;
  // Lanes along rows of C (time over that of lanes along columns, 20000 drawn products): column-major C 0.65 to 0.93; row-major, N <= 24,
  // 0.71 to 0.99 (139x1x7, 508 problems: 14.0 -> 9.3 us), N of 25 to 48 0.92 to 0.95 with two tiles per CU, 0.98 to 1.13 with more; at most a
  // tile per CU 0.83 to 0.99 whatever N is; else 1.0 to 1.33.
  const int64_t tiles = (int64_t)pl.grid.x * pl.grid.y * pl.grid.z;
  const bool rows = d.layout_c == GEMM_COL_MAJOR || tiles <= num_cus() || d.N <= (tiles <= 2 * num_cus() ? 48 : 24);
  auto go = [&](auto ak_c, auto bk_c) {
    constexpr bool AK = decltype(ak_c)::value, BK = decltype(bk_c)::value;
    if (rows) f32_any_kernel<AK, BK, MT, true><<<pl.grid, pl.block, 0, s>>>(r, a.c_si, a.c_sj);
    else f32_any_kernel<AK, BK, MT, false><<<pl.grid, pl.block, 0, s>>>(r, a.c_si, a.c_sj);
  };
  typedef std::true_type yes;
  typedef std::false_type no;
  if (ak && bk) go(yes(), yes());
  else if (ak) go(yes(), no());
  else if (bk) go(no(), yes());
  else go(no(), no());
  return hipGetLastError();
}

// the general matrix-core kernel in fp32 whatever the offsets are
hipError_t launch_f32_general(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  return launch_general_mfma_typed<float, float, 64, 64, 16>(pl, A, B, C, bias, s);
}

template <typename TIn, int TM, int TN, int TK>
hipError_t launch_general_mfma(const gemm_plan& pl, const void* A, const void* B, void* C,
                               const void* bias, hipStream_t s) {
  if constexpr (sizeof(TIn) == 4)
    if (f32_takes_any(pl.d, TM)) return launch_f32_any<TM>(pl, A, B, C, bias, s);
  if (pl.d.dtype_c == GEMM_F32)
    return launch_general_mfma_typed<TIn, float, TM, TN, TK>(pl, A, B, C, bias, s);
  return launch_general_mfma_typed<TIn, TIn, TM, TN, TK>(pl, A, B, C, bias, s);
}

// Does a float4 problem run on the kernel with slabs straight to LDS?  Its offsets inside a slab have to fit 32 bits.  And
// of its 64x64 tiles three fit a CU, four of the kernel that stages slabs through registers, which with a short K is ahead
// where it needs fewer rounds of the CUs for that: 3 to 4 tiles per CU, K <= 32 0.81 of the time (38x25 tiles, K = 12: 9.4
// against 12.0 us), 14x64 tiles with K = 64 / 128 / 192 1 / 1.27, 1 / 1.14, 1 / 1.07; 6 to 8 tiles per CU, K <= 32 0.90.  With
// as many rounds the slabs straight to LDS win, also with a K of one slab (one tile per CU 1.09, 4 to 6 1.04).
bool f32_takes_ring(const gemm_desc_t& d, int tile) {
  const int64_t lim = (int64_t)1 << 32, kMax = ((int64_t)1 << 31) - 512;
  if ((tile + 1) * d.lda * 4 >= lim || (tile + 1) * d.ldb * 4 >= lim || d.M >= kMax || d.N >= kMax || d.K >= kMax) return false;
  const double per_cu = (double)((d.M + 63) / 64) * (double)((d.N + 63) / 64) * d.batch / num_cus();
  const bool fewer_rounds = std::ceil(per_cu / 4) < std::ceil(per_cu / 3);
  return tile != 64 || !fewer_rounds || d.K > (per_cu <= 4 ? 192 : 32);
}

// fp32 operands in 16-byte pieces (the plan's extents and leading dimensions allow it: applicable()); pointers that
// are not 16-byte aligned take f32_any_kernel on the same grid, or the general kernel where offsets do not fit 32 bits
template <int TM, int TN>
hipError_t launch_f32_mfma(const gemm_plan& pl, const void* A, const void* B, void* C,
                           const void* bias, hipStream_t s) {
  const gemm_desc_t& d = pl.d;
  if (((uintptr_t)A & 15) || ((uintptr_t)B & 15)) {
    if (f32_takes_any(d, TM)) return launch_f32_any<TM>(pl, A, B, C, bias, s);
    return launch_general_mfma_typed<float, float, TM, TN, 16>(pl, A, B, C, bias, s);
  }
  const SimtArgs a = simt_args(pl, A, B, C, bias);
  const bool ak = d.layout_a == GEMM_ROW_MAJOR, bk = d.layout_b == GEMM_COL_MAJOR;   // K contiguous?
  if (f32_takes_ring(d, TM)) {
    constexpr int MT = TM / 64, S = f32_ring_stages(TM);
    MfmaArgs r = mfma16_args<TM, TN, false>(pl, A, B, C, bias);
    r.xcd_remap = d.batch == 1 || (r.tiles_m * (int64_t)r.tiles_n) % 8 == 0;
    if (ak && bk) f32_ring_kernel<true, true, MT, S><<<pl.grid, pl.block, 0, s>>>(r, a.c_si, a.c_sj);
    else if (ak) f32_ring_kernel<true, false, MT, S><<<pl.grid, pl.block, 0, s>>>(r, a.c_si, a.c_sj);
    else if (bk) f32_ring_kernel<false, true, MT, S><<<pl.grid, pl.block, 0, s>>>(r, a.c_si, a.c_sj);
    else f32_ring_kernel<false, false, MT, S><<<pl.grid, pl.block, 0, s>>>(r, a.c_si, a.c_sj);
    return hipGetLastError();
  }
  if (ak && bk) f32_mfma_kernel<true, true, TM, TN><<<pl.grid, pl.block, 0, s>>>(a);
  else if (ak) f32_mfma_kernel<true, false, TM, TN><<<pl.grid, pl.block, 0, s>>>(a);
  else if (bk) f32_mfma_kernel<false, true, TM, TN><<<pl.grid, pl.block, 0, s>>>(a);
  else f32_mfma_kernel<false, false, TM, TN><<<pl.grid, pl.block, 0, s>>>(a);
  return hipGetLastError();
}

// small fp32 problems: 16x16 tiles, K split over the waves of a workgroup; each K-contiguous operand
// is read in float4 groups when its extents, strides and pointer allow it
hipError_t launch_f32_small(const gemm_plan& pl, const void* A, const void* B, void* C,
                            const void* bias, hipStream_t s) {
  const gemm_desc_t& d = pl.d;
  F32SmallArgs a;
  a.g = simt_args(pl, A, B, C, bias);
  auto vec = [&](bool k_contiguous, int64_t ld, int64_t stride, const void* at) {
    if (!k_contiguous || d.K < 4) return 0;
    return d.K % 4 == 0 && ld % 4 == 0 && stride % 4 == 0 && ((uintptr_t)at & 15) == 0 ? 1 : 2;
  };
  a.vec_a = vec(d.layout_a == GEMM_ROW_MAJOR, d.lda, d.stride_a, A);
  a.vec_b = vec(d.layout_b == GEMM_COL_MAJOR, d.ldb, d.stride_b, B);
  // few rows of A of any alignment, a long K, B strided: value by value, where groups moved down by selects take 1.03 to 1.07 of the time
  // and up to 1.36 (42 problems of 1x16x2371 25.7 against 18.9 us; with nine rows, or a K up to 1024, 0.90 to 1.00)
  if (a.vec_a == 2 && a.vec_b == 0 && d.M <= 8 && d.K > 1024) a.vec_a = 0;
  if (a.vec_a == 2 || a.vec_b == 2) f32_small_kernel<true><<<pl.grid, pl.block, 0, s>>>(a);
  else f32_small_kernel<false><<<pl.grid, pl.block, 0, s>>>(a);
  return hipGetLastError();
}

// 16-bit operands of which at least one is not K-contiguous
template <typename T, int BM, int BN, int WM, int WN, int G, bool PERSIST, int S = 2>
hipError_t launch_mfma16t(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  const bool ak = pl.d.layout_a == GEMM_ROW_MAJOR, bk = pl.d.layout_b == GEMM_COL_MAJOR;
  if (ak) return launch_mfma16<T, T, BM, BN, WM, WN, G, PERSIST, true, false, S>(pl, A, B, C, bias, s);
  if (bk) return launch_mfma16<T, T, BM, BN, WM, WN, G, PERSIST, false, true, S>(pl, A, B, C, bias, s);
  return launch_mfma16<T, T, BM, BN, WM, WN, G, PERSIST, false, false, S>(pl, A, B, C, bias, s);
}
template <typename T, int BM, int BN, int WM, int WN, int KS, int NS>
hipError_t launch_ring_t(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  const bool ak = pl.d.layout_a == GEMM_ROW_MAJOR, bk = pl.d.layout_b == GEMM_COL_MAJOR;
  if (ak) return launch_ring<T, T, BM, BN, WM, WN, KS, NS, true, false>(pl, A, B, C, bias, s);
  if (bk) return launch_ring<T, T, BM, BN, WM, WN, KS, NS, false, true>(pl, A, B, C, bias, s);
  return launch_ring<T, T, BM, BN, WM, WN, KS, NS, false, false>(pl, A, B, C, bias, s);
}

template <typename TIn, int TM, int TN, int TK>
hipError_t launch_simt(const gemm_plan& pl, const void* A, const void* B, void* C,
                       const void* bias, hipStream_t s) {
  if (pl.d.dtype_c == GEMM_F32)
    return launch_simt_typed<TIn, float, TM, TN, TK>(pl, A, B, C, bias, s);
  return launch_simt_typed<TIn, TIn, TM, TN, TK>(pl, A, B, C, bias, s);
}

// the argument block every skinny kernel takes
SkinnyArgs skinny_args(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias) {
  const gemm_desc_t& d = pl.d;
  SkinnyArgs a;
  a.X = A; a.W = B; a.Y = C; a.bias = (const float*)bias;
  a.M = (int)d.M; a.N = (int)d.N; a.K = (int)d.K;
  a.ldx = d.lda; a.ldw = d.ldb; a.ldy = d.ldc;
  a.stride_x = d.stride_a; a.stride_w = d.stride_b; a.stride_y = d.stride_c;
  a.stride_bias = d.stride_bias;
  a.has_bias = epilogue_has_bias(d.epilogue);
  a.act = epilogue_activation(d.epilogue);
  a.scale = d.scale;
  a.y_f32 = d.dtype_c == GEMM_F32;
  return a;
}

template <typename T, int MB, int WAVES>
hipError_t launch_skinny(const gemm_plan& pl, const void* A, const void* B, void* C,
                         const void* bias, hipStream_t s) {
  skinny_gemm_kernel<T, MB, WAVES><<<pl.grid, pl.block, 0, s>>>(skinny_args(pl, A, B, C, bias));
  return hipGetLastError();
}

template <typename T, int DEPTH, int RB, int WAVES>
hipError_t launch_skinny_stage(const gemm_plan& pl, const void* A, const void* B, void* C,
                               const void* bias, hipStream_t s) {
  skinny_stage_kernel<T, DEPTH, RB, WAVES><<<pl.grid, pl.block, 0, s>>>(skinny_args(pl, A, B, C, bias));
  return hipGetLastError();
}

// Which problems does the built-in choice run on the kernel with x in registers (skinny_rows_kernel) instead of skinny_direct_kernel?  Measured on 166 drawn
// products (M 2 to 16, N 1024 to 130000, K 128 to 8192), its time over the other's: N <= 4096 (a panel per workgroup) 0.69 to 1.02
// with K > 1024, 1.1 to 1.5 with less (the start of a workgroup of eight waves, eight parts of K to add); N to 8192, where the
// panels of 32 rows are one round and those of 16 two, 0.90 to 0.96 with K of 3584 to 4096 (parts that fill two slabs, a little of x) and 0.97 to
// 1.23 otherwise; K <= 2048, where a panel is one slab, 0.89 to 1.24 up to N = 16384; everything else 0.77 to 1.06, 0.90 on average.
bool skinny_takes_rows(const gemm_desc_t& d) {
  if (d.N <= 16 * num_cus()) return true;
  if (d.N <= 32 * num_cus()) return d.K > 3584 && d.K <= 4096;
  return d.K > 2048 || d.N > 64 * num_cus();
}

template <typename T>
hipError_t launch_skinny_rows(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  const SkinnyArgs a = skinny_args(pl, A, B, C, bias);
  auto go = [&](auto slabs) {
    constexpr int S = decltype(slabs)::value;
    if (a.K == S * 2048) skinny_rows_kernel<T, S, true><<<pl.grid, pl.block, 0, s>>>(a);
    else skinny_rows_kernel<T, S, false><<<pl.grid, pl.block, 0, s>>>(a);
  };
  if (a.K > 6144) go(std::integral_constant<int, 4>());
  else if (a.K > 4096) go(std::integral_constant<int, 3>());
  else if (a.K > 2048) go(std::integral_constant<int, 2>());
  else go(std::integral_constant<int, 1>());
  return hipGetLastError();
}

template <typename T, int DEPTH, int RB, int WAVES>
hipError_t launch_skinny_direct(const gemm_plan& pl, const void* A, const void* B, void* C,
                                const void* bias, hipStream_t s) {
  skinny_direct_kernel<T, DEPTH, RB, WAVES><<<pl.grid, pl.block, 0, s>>>(skinny_args(pl, A, B, C, bias));
  return hipGetLastError();
}

// ---- the table of compiled instantiations ----------------------------------------------

#define SIMT_CFG(TM, TN, TK)                                                               \
  { "simt_" #TM "x" #TN "x" #TK, KIND_SIMT, TM, TN, TK, 256,                               \
    (int)(sizeof(float) * TK * (TM + 4 + TN + 4)),                                         \
    { launch_simt<float, TM, TN, TK>, launch_simt<bf16_t, TM, TN, TK>,                     \
      launch_simt<f16_t, TM, TN, TK> } }

// the general kernel on the matrix cores (fp32 MFMA): same problems, same grid as SIMT_CFG
#define GENERAL_MFMA_CFG(TM, TN, TK)                                                       \
  { "general_mfma32_" #TM "x" #TN "x" #TK, KIND_SIMT, TM, TN, TK, 256,                     \
    (int)(sizeof(float) * TK * (TM + 4 + TN + 4)),                                         \
    { launch_general_mfma<float, TM, TN, TK>, launch_general_mfma<bf16_t, TM, TN, TK>,     \
      launch_general_mfma<f16_t, TM, TN, TK> }, 5 }

// fp32 operands and output moved as float4 groups, slabs of 32 columns of K
#define F32_MFMA_CFG(TM, TN)                                                               \
  { "f32mfma_" #TM "x" #TN "x32", KIND_F32_VEC, TM, TN, kF32TileK, 256,                    \
    f32_ring_stages(TM) * (TM + TN) * 128,                                                 \
    { launch_f32_mfma<TM, TN>, nullptr, nullptr } }

// small fp32 problems: 16x16 tiles, 256 columns of K per round of the four waves
#define F32_SMALL_CFG()                                                                    \
  { "f32small_16x16x256", KIND_SIMT, 16, 16, 256, 256, 4096, { launch_f32_small, nullptr, nullptr } }

// general_mfma32_64x64x16 in fp32 where its offsets would allow f32_any_kernel, too
#define F32_GENERAL_CFG()                                                                  \
  { "f32general_64x64x16", KIND_SIMT, 64, 64, 16, 256, (int)(sizeof(float) * 16 * (64 + 4 + 64 + 4)), { launch_f32_general, nullptr, nullptr } }

#define MFMA_CFG(BM, BN, BK, WM, WN, NS)                                                   \
  { "mfma_" #BM "x" #BN "x" #BK "_w" #WM "x" #WN "_s" #NS, KIND_MFMA, BM, BN, BK,          \
    64 * WM * WN, MfmaTile<bf16_t, BM, BN, BK, WM, WN, NS>::LDS_BYTES,                     \
    { nullptr, launch_mfma<bf16_t, bf16_t, BM, BN, BK, WM, WN, NS>,                        \
      launch_mfma<f16_t, f16_t, BM, BN, BK, WM, WN, NS> } }
// the same product on the 16x16x32 MFMA shape (slabs of 64 columns of K, two stages)
#define MFMA16_CFG(BM, BN, WM, WN, G)                                                      \
  { "mfma16_" #BM "x" #BN "x64_w" #WM "x" #WN, KIND_MFMA, BM, BN, 64,                      \
    64 * WM * WN, Mfma16Tile<bf16_t, BM, BN, WM, WN, G>::LDS_BYTES +                       \
                      Mfma16Tile<bf16_t, BM, BN, WM, WN, G>::DUMP_BYTES,                   \
    { nullptr, launch_mfma16<bf16_t, bf16_t, BM, BN, WM, WN, G, false>,                    \
      launch_mfma16<f16_t, f16_t, BM, BN, WM, WN, G, false> }, 0 }
// persistent workgroups (K a whole number of slabs, at least two): the grid is the number of
// workgroups the chip holds at once, each walks over its share of the tiles
#define MFMA16P_CFG(BM, BN, WM, WN, G)                                                     \
  { "mfma16_" #BM "x" #BN "x64_w" #WM "x" #WN "_p", KIND_MFMA, BM, BN, 64,                 \
    64 * WM * WN, Mfma16Tile<bf16_t, BM, BN, WM, WN, G>::LDS_BYTES +                       \
                      Mfma16Tile<bf16_t, BM, BN, WM, WN, G>::EPI_BYTES,                    \
    { nullptr, launch_mfma16<bf16_t, bf16_t, BM, BN, WM, WN, G, true>,                     \
      launch_mfma16<f16_t, f16_t, BM, BN, WM, WN, G, true> }, 1 }
// either of the two for operands whose K is not contiguous (P: 0 = one tile per workgroup, 1 = persistent)
#define MFMA16T_CFG(SUFFIX, BM, BN, WM, WN, G, P)                                           \
  { "mfma16t_" #BM "x" #BN "x64_w" #WM "x" #WN SUFFIX, KIND_MFMA_T, BM, BN, 64,             \
    64 * WM * WN, Mfma16Tile<bf16_t, BM, BN, WM, WN, G, 2, false>::LDS_BYTES +             \
                      (P ? Mfma16Tile<bf16_t, BM, BN, WM, WN, G>::EPI_BYTES                \
                         : Mfma16Tile<bf16_t, BM, BN, WM, WN, G>::DUMP_BYTES),             \
    { nullptr, launch_mfma16t<bf16_t, BM, BN, WM, WN, G, P != 0>,                          \
      launch_mfma16t<f16_t, BM, BN, WM, WN, G, P != 0> }, P }
// fp8 (E4M3) operands, bf16 or fp32 output: the same slabs in bytes (BK is twice as many values)
// (persistent workgroups where K is a whole number of slabs, at least two; one tile per workgroup otherwise)
template <int BM, int BN, int WM, int WN, int G>
hipError_t launch_mfma16f8(const gemm_plan& pl, const void* A, const void* B, void* C, const void* bias, hipStream_t s) {
  if (persists(*pl.cfg, pl.d)) return launch_mfma16<f8e4m3_t, bf16_t, BM, BN, WM, WN, G, true>(pl, A, B, C, bias, s);
  return launch_mfma16<f8e4m3_t, bf16_t, BM, BN, WM, WN, G, false>(pl, A, B, C, bias, s);
}
#define MFMA16F8_CFG(BM, BN, WM, WN, G)                                                    \
  { "mfma8_" #BM "x" #BN "x128_w" #WM "x" #WN "_s2", KIND_MFMA, BM, BN, 128, 64 * WM * WN, \
    Mfma16Tile<f8e4m3_t, BM, BN, WM, WN, G>::LDS_BYTES + Mfma16Tile<f8e4m3_t, BM, BN, WM, WN, G>::EPI_BYTES, \
    { nullptr, nullptr, nullptr, launch_mfma16f8<BM, BN, WM, WN, G> }, 2 }
// one tile per workgroup whatever K is
#define MFMA16F8_ONE_CFG(BM, BN, WM, WN, G)                                                \
  { "mfma8_" #BM "x" #BN "x128_w" #WM "x" #WN "_one", KIND_MFMA, BM, BN, 128, 64 * WM * WN, \
    Mfma16Tile<f8e4m3_t, BM, BN, WM, WN, G>::LDS_BYTES + Mfma16Tile<f8e4m3_t, BM, BN, WM, WN, G>::DUMP_BYTES, \
    { nullptr, nullptr, nullptr, launch_mfma16<f8e4m3_t, bf16_t, BM, BN, WM, WN, G, false> }, 0 }

// bn = workgroups per CU the grid is sized for
#define SKINNY_CFG(MB, WAVES, PER_CU)                                                      \
  { "skinny_m" #MB "_w" #WAVES "_g" #PER_CU, KIND_SKINNY, MB, PER_CU, kSkinnyKC,           \
    64 * WAVES, (MB == 1 || (MB == 2 && WAVES <= 4)) ? 16 : MB * kSkinnyKC * 2,            \
    { nullptr, launch_skinny<bf16_t, MB, WAVES>, launch_skinny<f16_t, MB, WAVES> } }

// skinny on the matrix cores, W staged through registers into wave-private LDS slabs:
// bm = 16 x rows, bn = 32 rows of W per workgroup, bk = k per slab
#define SKINNY_STAGE_CFG(DEPTH, RB)                                                        \
  { "skinnystage_d" #DEPTH "_b" #RB, KIND_SKINNY_PANEL, 16, 32, RB / 2, 256, 4 * 48 * RB,     \
    { nullptr, launch_skinny_stage<bf16_t, DEPTH, RB, 4>, launch_skinny_stage<f16_t, DEPTH, RB, 4> } }
// skinny with W staged through LDS and x fragments straight from L2 (16x16x32 MFMA): same panel shape
#define SKINNY_DIRECT_CFG(DEPTH, RB, WAVES)                                                \
  { "skinnydirect_d" #DEPTH "_b" #RB "_w" #WAVES, KIND_SKINNY_PANEL, 16, 32, RB / 2, 64 * WAVES, WAVES * 32 * RB, \
    { nullptr, launch_skinny_direct<bf16_t, DEPTH, RB, WAVES>, launch_skinny_direct<f16_t, DEPTH, RB, WAVES> } }
// the same with x in registers and panels of 16 rows of W
#define SKINNY_ROWS_CFG()                                                                  \
  { "skinnydirect_d2_b512_w4_rows", KIND_SKINNY_PANEL, 16, kSkinnyRowsPanel, 256, 512, kSkinnyRowsLds, \
    { nullptr, launch_skinny_rows<bf16_t>, launch_skinny_rows<f16_t> }, 3 }
// 128x128 tiles with four slabs in LDS, one workgroup per CU
#define MFMA16S_CFG(BM, BN, WM, WN, G, S)                                                  \
  { "mfma16_" #BM "x" #BN "x64_w" #WM "x" #WN "_s" #S, KIND_MFMA, BM, BN, 64, 64 * WM * WN, \
    Mfma16Tile<bf16_t, BM, BN, WM, WN, G, S>::LDS_BYTES,                                   \
    { nullptr, launch_mfma16<bf16_t, bf16_t, BM, BN, WM, WN, G, false, true, true, S>,     \
      launch_mfma16<f16_t, f16_t, BM, BN, WM, WN, G, false, true, true, S> }, 0, 0.33f, 0.0f },
#define MFMA16F8S_CFG(BM, BN, WM, WN, G, S)                                                \
  { "mfma8_" #BM "x" #BN "x128_w" #WM "x" #WN "_s" #S, KIND_MFMA, BM, BN, 128, 64 * WM * WN, \
    Mfma16Tile<f8e4m3_t, BM, BN, WM, WN, G, S>::LDS_BYTES,                                 \
    { nullptr, nullptr, nullptr, launch_mfma16<f8e4m3_t, bf16_t, BM, BN, WM, WN, G, false, true, true, S> }, 0, 0.33f, 0.0f },
#define MFMA16TS_CFG(BM, BN, WM, WN, G, S)                                                 \
  { "mfma16t_" #BM "x" #BN "x64_w" #WM "x" #WN "_s" #S, KIND_MFMA_T, BM, BN, 64, 64 * WM * WN, \
    Mfma16Tile<bf16_t, BM, BN, WM, WN, G, S>::LDS_BYTES,                                   \
    { nullptr, launch_mfma16t<bf16_t, BM, BN, WM, WN, G, false, S>,                        \
      launch_mfma16t<f16_t, BM, BN, WM, WN, G, false, S> }, 0, 0.33f, 0.0f },
// small tiles, slabs of K in a ring
#define RING_ENTRY(NAME, KIND, T, BM, BN, WM, WN, KS, NS, T1, T2, ...)                     \
  { NAME "_" #BM "x" #BN "_k" #KS "_w" #WM "x" #WN "_s" #NS, KIND, BM, BN, RingTile<T, BM, BN, WM, WN, KS, NS>::BK, \
    64 * WM * WN, RingTile<T, BM, BN, WM, WN, KS, NS>::LDS_BYTES, { nullptr, __VA_ARGS__ }, 0, T1##f, T2##f },
#define RING_CFG(BM, BN, WM, WN, KS, NS, T1, T2)                                           \
  RING_ENTRY("mfma16", KIND_MFMA, bf16_t, BM, BN, WM, WN, KS, NS, T1, T2,                  \
             launch_ring<bf16_t, bf16_t, BM, BN, WM, WN, KS, NS, true, true>,              \
             launch_ring<f16_t, f16_t, BM, BN, WM, WN, KS, NS, true, true>)
#define RINGT_CFG(BM, BN, WM, WN, KS, NS, T1, T2)                                          \
  RING_ENTRY("mfma16t", KIND_MFMA_T, bf16_t, BM, BN, WM, WN, KS, NS, T1, T2,               \
             launch_ring_t<bf16_t, BM, BN, WM, WN, KS, NS>, launch_ring_t<f16_t, BM, BN, WM, WN, KS, NS>)
#define RING8_CFG(BM, BN, WM, WN, KS, NS, T1, T2)                                          \
  RING_ENTRY("mfma8", KIND_MFMA, f8e4m3_t, BM, BN, WM, WN, KS, NS, T1, T2, nullptr, nullptr, \
             launch_ring<f8e4m3_t, bf16_t, BM, BN, WM, WN, KS, NS, true, true>)
// small tiles, K split over the waves
#define KSPLIT_CFG(BM, BN, W, NS, T1)                                                      \
  { "ksplit16_" #BM "x" #BN "_w" #W "_s" #NS, KIND_MFMA, BM, BN, 64, 64 * W, kSplitLds<BM, BN, W, NS>, \
    { nullptr, launch_ksplit<bf16_t, BM, BN, W, NS>, launch_ksplit<f16_t, BM, BN, W, NS> }, 4, T1##f, 0.0f },
// 16-bit operands of any alignment, two slabs
#define MFMA16G_CFG(BM, BN, WM, WN, KS, T1, T2)                                            \
  { "mfma16g_" #BM "x" #BN "_k" #KS "_w" #WM "x" #WN, KIND_MFMA_G, BM, BN, KS * 64, 64 * WM * WN, \
    RingTile<bf16_t, BM, BN, WM, WN, KS, 2>::LDS_BYTES,                                    \
    { nullptr, launch_mfma16g<bf16_t, BM, BN, WM, WN, KS>, launch_mfma16g<f16_t, BM, BN, WM, WN, KS> }, 0, T1##f, T2##f },
const Config kConfigs[] = {
    SIMT_CFG(64, 64, 16),
    SIMT_CFG(32, 32, 16),
    SIMT_CFG(32, 32, 64),
    MFMA16P_CFG(256, 256, 2, 4, 2),
    MFMA16P_CFG(128, 128, 2, 2, 2),
    MFMA16_CFG(256, 256, 2, 4, 2),
    MFMA16_CFG(256, 256, 2, 2, 2),
    MFMA16_CFG(128, 128, 2, 2, 2),
    MFMA_CFG(256, 256, 64, 2, 4, 2),
    MFMA_CFG(256, 256, 64, 2, 2, 2),
    MFMA_CFG(256, 128, 64, 2, 2, 2),
    MFMA_CFG(128, 128, 64, 2, 2, 2),
    MFMA_CFG(256, 192, 64, 4, 2, 2),
    MFMA16F8_CFG(256, 256, 2, 4, 4),
    MFMA16F8_CFG(128, 128, 2, 2, 4),
    MFMA16F8_CFG(256, 192, 4, 2, 4),
    MFMA16F8_CFG(224, 256, 2, 4, 4),
    MFMA16F8_CFG(192, 256, 2, 4, 4),
    MI355GEMM_MFMA16F8S_TILES(MFMA16F8S_CFG)
    F32_MFMA_CFG(128, 128),
    F32_MFMA_CFG(64, 64),
    F32_SMALL_CFG(),
    GENERAL_MFMA_CFG(128, 128, 16),
    GENERAL_MFMA_CFG(64, 64, 16),
    SKINNY_CFG(1, 4, 1),
    SKINNY_CFG(2, 4, 1),
    SKINNY_CFG(4, 4, 1),
    SKINNY_CFG(8, 4, 1),
    SKINNY_CFG(1, 8, 1),
    SKINNY_CFG(1, 8, 2),
    SKINNY_CFG(2, 8, 1),
    SKINNY_CFG(4, 8, 1),
    SKINNY_STAGE_CFG(3, 256),
    SKINNY_STAGE_CFG(2, 512),
    SKINNY_DIRECT_CFG(2, 512, 4),
    SKINNY_DIRECT_CFG(3, 512, 4),
    SKINNY_DIRECT_CFG(2, 256, 8),
    MFMA16T_CFG("_p", 256, 256, 2, 4, 2, 1),
    MFMA16T_CFG("_p", 128, 128, 2, 2, 2, 1),
    MFMA16T_CFG("", 256, 256, 2, 4, 2, 0),
    MFMA16T_CFG("", 128, 128, 2, 2, 2, 0),
    MFMA16P_CFG(224, 256, 2, 4, 2),
    MFMA16P_CFG(192, 256, 2, 4, 2),
    MFMA16_CFG(224, 256, 2, 4, 2),
    MFMA16_CFG(192, 256, 2, 4, 2),
    MFMA16T_CFG("_p", 192, 256, 2, 4, 2, 1),
    MFMA16T_CFG("", 192, 256, 2, 4, 2, 0),
    MI355GEMM_MFMA16S_TILES(MFMA16S_CFG)
    MI355GEMM_MFMA16S_TILES(MFMA16TS_CFG)
    MI355GEMM_RINGS(RING_CFG)
    MI355GEMM_RINGS16(RING_CFG)
    MI355GEMM_KSPLITS(KSPLIT_CFG)
    MI355GEMM_RINGS_T(RINGT_CFG)
    MI355GEMM_RINGS(RING8_CFG)
    MI355GEMM_MFMA16G_TILES(MFMA16G_CFG)
    MFMA16F8_ONE_CFG(256, 256, 2, 4, 4),
    MFMA16F8_ONE_CFG(128, 128, 2, 2, 4),
    MFMA16F8_ONE_CFG(256, 192, 4, 2, 4),
    MFMA16F8_ONE_CFG(224, 256, 2, 4, 4),
    MFMA16F8_ONE_CFG(192, 256, 2, 4, 4),
    F32_GENERAL_CFG(),
    SKINNY_ROWS_CFG(),
};
constexpr int kNumConfigs = (int)(sizeof(kConfigs) / sizeof(kConfigs[0]));

// Compute units of the device the plans are made for: asked of the runtime once (the current
// device at the first plan); 256, an MI355X, where no device can be asked (plans can be made
// and inspected on a machine without a GPU).
int num_cus() {
  static const int n = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
      return cus;
    (void)hipGetLastError();
    return 256;
  }();
  return n;
}

// ---- validation -----------------------------------------------------------------------

bool in_range(int v, int lo, int hi) { return v >= lo && v <= hi; }

// Resolve packed (0) leading dimensions / strides and check every field.
int resolve(const gemm_desc_t* in, gemm_desc_t* out) {
  gemm_desc_t d = *in;
  if (!in_range(d.layout_a, 0, 1) || !in_range(d.layout_b, 0, 1) || !in_range(d.layout_c, 0, 1) ||
      !in_range(d.dtype_a, 0, 3) || !in_range(d.dtype_b, 0, 3) || !in_range(d.dtype_c, 0, 3) ||
      !in_range(d.dtype_bias, 0, 2) || !in_range(d.epilogue, 0, GEMM_EPI_SIGMOID_SCALE_RESIDUAL))
    return GEMM_ERR_BAD_ENUM;
  if (epilogue_has_scale(d.epilogue)) {
    if (!std::isfinite(d.scale)) return GEMM_ERR_BAD_SCALE;
  } else {
    d.scale = 1.0f;                              // ignored: keep the plan's copy tidy
  }
  if (d.M <= 0 || d.N <= 0 || d.K <= 0 || d.batch < 1) return GEMM_ERR_BAD_DIM;
  const int64_t kMaxDim = (int64_t)1 << 30;
  if (d.M > kMaxDim || d.N > kMaxDim || d.K > kMaxDim || d.batch > 65535) return GEMM_ERR_BAD_DIM;
  if (d.lda < 0 || d.ldb < 0 || d.ldc < 0 || d.stride_a < 0 || d.stride_b < 0 ||
      d.stride_c < 0 || d.stride_bias < 0)
    return GEMM_ERR_BAD_LD;

  const int64_t a_minor = d.layout_a == GEMM_ROW_MAJOR ? d.K : d.M;
  const int64_t a_major = d.layout_a == GEMM_ROW_MAJOR ? d.M : d.K;
  const int64_t b_minor = d.layout_b == GEMM_ROW_MAJOR ? d.N : d.K;
  const int64_t b_major = d.layout_b == GEMM_ROW_MAJOR ? d.K : d.N;
  const int64_t c_minor = d.layout_c == GEMM_ROW_MAJOR ? d.N : d.M;
  const int64_t c_major = d.layout_c == GEMM_ROW_MAJOR ? d.M : d.N;
  if (d.lda == 0) d.lda = a_minor;
  if (d.ldb == 0) d.ldb = b_minor;
  if (d.ldc == 0) d.ldc = c_minor;
  if (d.lda < a_minor || d.ldb < b_minor || d.ldc < c_minor) return GEMM_ERR_BAD_LD;
  const int64_t kMaxLd = (int64_t)1 << 40;
  if (d.lda > kMaxLd || d.ldb > kMaxLd || d.ldc > kMaxLd) return GEMM_ERR_BAD_LD;
  // extents in elements: major * ld must stay below 2^62 (no signed overflow anywhere below)
  int64_t a_full, b_full, c_full;
  const int64_t kMaxSpan = (int64_t)1 << 62;
  if (__builtin_mul_overflow(a_major, d.lda, &a_full) || a_full >= kMaxSpan ||
      __builtin_mul_overflow(b_major, d.ldb, &b_full) || b_full >= kMaxSpan ||
      __builtin_mul_overflow(c_major, d.ldc, &c_full) || c_full >= kMaxSpan)
    return GEMM_ERR_BAD_LD;
  const int64_t a_span = a_full - d.lda + a_minor;
  const int64_t b_span = b_full - d.ldb + b_minor;
  const int64_t c_span = c_full - d.ldc + c_minor;
  if (d.stride_a == 0) d.stride_a = a_full;
  if (d.stride_b == 0) d.stride_b = b_full;
  if (d.stride_c == 0) d.stride_c = c_full;
  if (d.batch > 1) {
    // Reading one A or B slab for several batches would be legal, but the stride
    // field uses 0 for "packed", so overlapping inputs are not expressible; an
    // overlapping output is always an error.
    if (d.stride_a < a_span || d.stride_b < b_span || d.stride_c < c_span) return GEMM_ERR_BAD_LD;
    if (d.stride_bias != 0 && d.stride_bias < d.N) return GEMM_ERR_BAD_LD;
  }
  if (d.dtype_a != d.dtype_b) return GEMM_ERR_UNSUPPORTED;
  if (d.dtype_a == GEMM_F8E4M3) {
    if (d.dtype_c != GEMM_BF16 && d.dtype_c != GEMM_F32) return GEMM_ERR_UNSUPPORTED;
  } else if (d.dtype_c != d.dtype_a && d.dtype_c != GEMM_F32) {
    return GEMM_ERR_UNSUPPORTED;
  }
  if (d.dtype_bias != GEMM_F32) return GEMM_ERR_UNSUPPORTED;
  *out = d;
  return GEMM_OK;
}

// The alignment the tiled 16-bit and fp8 kernels need: every operand's contiguous extent, leading dimension and
// batch stride a whole number of 16-byte pieces (and C row-major).
bool whole_pieces(const gemm_desc_t& d) {
  const int64_t epc = 16 / esize(d.dtype_a);
  const bool ak = d.layout_a == GEMM_ROW_MAJOR, bk = d.layout_b == GEMM_COL_MAJOR;
  return d.layout_c == GEMM_ROW_MAJOR && (ak ? d.K : d.M) % epc == 0 && (bk ? d.K : d.N) % epc == 0 &&
         d.lda % epc == 0 && d.ldb % epc == 0 && d.stride_a % epc == 0 && d.stride_b % epc == 0;
}

// Can instantiation c run problem d?
bool applicable(const Config& c, const gemm_desc_t& d) {
  if (!c.launch[d.dtype_a]) return false;
  if (c.kind == KIND_SIMT) return true;
  if (c.kind == KIND_F32_VEC) {
    // float4 groups along the contiguous index of A and of B: extents, leading dimensions and batch
    // strides in multiples of 4 elements; fp32 result
    const bool ak = d.layout_a == GEMM_ROW_MAJOR, bk = d.layout_b == GEMM_COL_MAJOR;
    return d.dtype_c == GEMM_F32 && d.lda % 4 == 0 && d.ldb % 4 == 0 && d.stride_a % 4 == 0 &&
           d.stride_b % 4 == 0 && (ak ? d.K : d.M) % 4 == 0 && (bk ? d.K : d.N) % 4 == 0;
  }
  if (c.kind == KIND_MFMA_G) {
    // what the tiled kernels do not take; the row limit is that of the general kernels' grids, 32-bit lane offsets
    const bool ak = d.layout_a == GEMM_ROW_MAJOR, bk = d.layout_b == GEMM_COL_MAJOR;
    const int64_t kMax = ((int64_t)1 << 31) - 512, lim = (int64_t)1 << 32;
    const int64_t a_rows = ak ? c.bm : c.bk + 1, b_rows = bk ? c.bn : c.bk + 1;
    const int64_t tiles = ((d.M + c.bm - 1) / c.bm) * ((d.N + c.bn - 1) / c.bn);
    return !whole_pieces(d) && d.M <= 65535 * 32 && d.N < kMax && d.K < kMax && a_rows * d.lda * 2 < lim &&
           b_rows * d.ldb * 2 < lim && tiles * d.batch < ((int64_t)1 << 31);
  }
  if (c.kind == KIND_MFMA_T) {
    // Row-major C, at least one operand not K-contiguous; 16-byte pieces along each operand's contiguous
    // index (its extent, leading dimension and batch stride multiples of 8), 32-bit lane offsets inside a slab.
    const bool ak = d.layout_a == GEMM_ROW_MAJOR, bk = d.layout_b == GEMM_COL_MAJOR;
    if ((ak && bk) || !whole_pieces(d)) return false;
    const int64_t kMax = ((int64_t)1 << 31) - 512;
    if (d.M >= kMax || d.N >= kMax || d.K >= kMax) return false;
    const int64_t a_rows = ak ? c.bm : c.bk + 1, b_rows = bk ? c.bn : c.bk + 1;
    if (a_rows * d.lda * 2 >= ((int64_t)1 << 32) || b_rows * d.ldb * 2 >= ((int64_t)1 << 32)) return false;
    if (c.persist == 1 && (d.K % c.bk != 0 || d.K < 2 * c.bk)) return false;
    const int64_t tiles = ((d.M + c.bm - 1) / c.bm) * ((d.N + c.bn - 1) / c.bn);
    return (persists(c, d) || c.t1 > 0 ? tiles * d.batch : tiles) < ((int64_t)1 << 31);
  }
  // The MFMA and skinny kernels take K-contiguous A and B, row-major C, and move
  // 16-byte pieces: every row start must be 16-byte aligned.
  if (d.layout_a != GEMM_ROW_MAJOR || d.layout_b != GEMM_COL_MAJOR || d.layout_c != GEMM_ROW_MAJOR)
    return false;
  const int64_t epc = 16 / esize(d.dtype_a);                 // operand elements per 16-byte piece
  if (d.K % epc || d.lda % epc || d.ldb % epc || d.stride_a % epc || d.stride_b % epc) return false;
  if (d.M >= ((int64_t)1 << 31) - 512 || d.N >= ((int64_t)1 << 31) - 512 ||
      d.K >= ((int64_t)1 << 31) - 512)
    return false;
  if (c.kind == KIND_SKINNY) return d.M <= c.bm;
  // (x in registers: one problem, a whole panel, what the registers hold; up to K = 1024 it is 1.1 to 1.5 behind: skinny_takes_rows)
  if (c.persist == 3 && (d.batch != 1 || d.N < c.bn || d.K <= 1024 || d.K > kSkinnyRowsMaxK)) return false;
  if (c.kind == KIND_SKINNY_PANEL)   // 32-bit lane offsets inside a 32-row panel
    return d.M <= c.bm && 32 * d.ldb * 2 < ((int64_t)1 << 32) && 32 * d.lda * 2 < ((int64_t)1 << 32) &&
           (d.N + 31) / 32 < ((int64_t)1 << 31);
  // MFMA: per-lane byte offsets inside a tile's row panel are 32-bit.
  if ((int64_t)c.bm * d.lda * esize(d.dtype_a) >= ((int64_t)1 << 32) ||
      (int64_t)c.bn * d.ldb * esize(d.dtype_a) >= ((int64_t)1 << 32))
    return false;
  if (c.persist == 1 && (d.K % c.bk != 0 || d.K < 2 * c.bk)) return false;   // whole slabs, at least two
  if (c.persist == 4 && (d.lda % 64 != 0 || d.ldb % 64 != 0)) return false;  // rows on 128-byte lines (weighs_ksplit)
  const int64_t tiles = ((d.M + c.bm - 1) / c.bm) * ((d.N + c.bn - 1) / c.bn);
  return (persists(c, d) || c.t1 > 0 ? tiles * d.batch : tiles) < ((int64_t)1 << 31);
}

// LDS bytes and K step of the kernel a plan runs for 16-byte aligned operands
struct Runs { int lds, bk; };
Runs plan_runs(const gemm_plan& pl) {
  const Config& c = *pl.cfg;
  const gemm_desc_t& d = pl.d;
  if (c.persist == 2 && !persists(c, d)) return {2 * (c.bm + c.bn) * 128 + (c.threads == 512 ? 256 : 0), c.bk};   // (no staging area)
  if (c.persist == 5 && f32_takes_any(d, c.bm)) return {2 * 2 * c.bm * 128, kF32TileK};                            // f32_any_kernel
  if (c.kind != KIND_F32_VEC || f32_takes_ring(d, c.bm)) return {c.lds_bytes, c.bk};
  return {f32_mfma_lds(c.bm, d.layout_a == GEMM_ROW_MAJOR) + f32_mfma_lds(c.bm, d.layout_b == GEMM_COL_MAJOR), c.bk};
}

int find_config(const char* name) {
  for (int i = 0; i < kNumConfigs; ++i)
    if (!std::strcmp(kConfigs[i].name, name)) return i;
  return -1;
}

// Cost models of one MFMA tile shape on an M x N x K (x batch) problem, in microseconds.
//
// tile_cost, fp8 operands, and 16-bit ones on tiles of 64x64 and larger: a launch, and as many turns of the workgroups that the chip holds at once
// as there are tiles for, each of `tile` us (first loads, C) and `slab` us per slab, a fifth more per operand whose rows do not start
// on 128-byte lines, and more for fp32 results; a turn that fills the chip to f takes part + (1 - part) f of a full one.  At the
// other end the bytes of A, B and C.  Fitted to the times of 16000 drawn products (K from 32 to 16384, batches, all layouts, operands
// from HBM; those within 30 % of the fastest): 11 % rms for each of these kernels.  Against the fastest kernel the choice costs on
// average 2.0 % for K of 64 to 768, 0.5 % for one to five rounds of 256x256 tiles, 1.0 % for other layers, 2.1 % for batches and
// 2.5 % for those with a K up to 8192 (with constants fitted to a long K, a step at K = 512 and no part turns for 128x128 tiles it
// was 3.9, 0.9, 1.8, 3.8 and 2.9 %: 202 x (387x104x32) 10.4 us, 19.2 so).  (Two slab times by hand, 1.340 and 1.000 for 1.284 and 0.968: of
// 43 products that took 224-row tiles with one tile per workgroup, 192-row ones were 6 to 7 % faster.)
// fp8: from such a fit, then moved so that the choice is as near as possible to the fastest kernel over 60 % of 15768 drawn products (M from
// 16, N and K from 64; both result types, batches): 1.78 % from it on the other 40 % (as fitted 2.3; so its microseconds are those of a
// comparison, the launch among them).  Against the kernels on the 32x32x64 instruction with their own choice 0.975; of the products with a K
// of 256 to 1023 and fp32 results 0.994, 39 of 2172 more than 10 % slower, about what two measurements of one kernel differ.
struct SharedTimes { double launch, off_line, apart, f32, operands, c32, c16; };   // us; shares of a slab; us; TB/s
const SharedTimes kShared16 = {2.8, 0.171, 0.26, 1.5, 3.68, 4.24, 2.22}, kShared8 = {1.07, 0.182, 0.342, 1.05, 8.32, 6.68, 5.82};
struct TileTimes { const char* name; double tile, slab, part; };
const TileTimes kTileTimes[] = {
    {"mfma16_128x128x64_w2x2", 3.77, 0.959, 0.53}, {"mfma16_128x128x64_w2x2_p", 3.30, 0.956, 0.61}, {"mfma16_128x128x64_w2x2_s4", 3.16, 0.531, 0.78},
    {"mfma16_192x256x64_w2x4", 5.76, 1.217, 0.62}, {"mfma16_192x256x64_w2x4_p", 5.10, 1.151, 0.71}, {"mfma16_224x256x64_w2x4", 6.54, 1.340, 0.65},
    {"mfma16_224x256x64_w2x4_p", 6.05, 1.274, 0.66}, {"mfma16_256x256x64_w2x2", 9.53, 1.477, 0.67}, {"mfma16_256x256x64_w2x4", 7.98, 1.456, 0.57},
    {"mfma16_256x256x64_w2x4_p", 6.92, 1.445, 0.59}, {"mfma16_64x64_k1_w2x4_s5", 1.87, 0.473, 0.36}, {"mfma16_64x64_k2_w2x4_s4", 1.41, 0.546, 0.60},
    {"mfma16t_128x128x64_w2x2", 3.08, 0.905, 0.50}, {"mfma16t_128x128x64_w2x2_p", 2.61, 0.929, 0.57}, {"mfma16t_128x128x64_w2x2_s4", 2.85, 0.501, 0.69},
    {"mfma16t_192x256x64_w2x4", 6.04, 1.085, 0.55}, {"mfma16t_192x256x64_w2x4_p", 4.62, 1.031, 0.73}, {"mfma16t_256x256x64_w2x4", 8.38, 1.279, 0.53},
    {"mfma16t_256x256x64_w2x4_p", 6.34, 1.246, 0.61}, {"mfma16t_64x64_k1_w2x4_s5", 1.51, 0.507, 0.37}, {"mfma16t_64x64_k2_w2x4_s4", 1.14, 0.583, 0.63},
    {"ksplit16_64x64_w8_s1", 1.41, 0.235, 0.60},        // (0.86 of the time of the ring's tile, for half its slab)
    {"mfma_128x128x64_w2x2_s2", 4.48, 1.000, 0.50}, {"mfma_256x128x64_w2x2_s2", 5.67, 0.993, 0.82}, {"mfma_256x192x64_w4x2_s2", 6.16, 1.271, 0.62},
    {"mfma_256x256x64_w2x4_s2", 8.48, 1.521, 0.55},
    {"mfma_256x256x64_w2x2_s2", 8.48, 1.521, 0.55},     // (not timed: as the shape with eight waves, which goes first)
    {"mfma8_128x128x128_w2x2_s2", 2.70, 0.890, 0.71}, {"mfma8_128x128x128_w2x2_s4", 2.88, 0.512, 0.68},
    {"mfma8_192x256x128_w2x4_s2", 4.13, 1.096, 0.72}, {"mfma8_224x256x128_w2x4_s2", 5.53, 1.042, 0.72},
    {"mfma8_256x192x128_w4x2_s2", 3.69, 1.018, 0.84}, {"mfma8_256x256x128_w2x4_s2", 6.26, 1.168, 0.70},
    {"mfma8_32x32_k2_w2x2_s4", 1.14, 0.402, 0.81}, {"mfma8_32x32_k4_w2x2_s3", 0.81, 0.488, 0.68}, {"mfma8_64x32_k2_w4x2_s4", 1.54, 0.307, 0.82},
    {"mfma8_64x64_k1_w2x4_s5", 1.92, 0.405, 0.58}, {"mfma8_64x64_k2_w2x4_s4", 1.77, 0.528, 0.72}, {"mfma8_128x128x128_w2x2_one", 3.51, 0.838, 0.69},
    {"mfma8_192x256x128_w2x4_one", 6.53, 1.154, 0.57}, {"mfma8_224x256x128_w2x4_one", 8.72, 1.142, 0.61},
    {"mfma8_256x192x128_w4x2_one", 7.74, 1.020, 0.70}, {"mfma8_256x256x128_w2x4_one", 9.96, 1.281, 0.54},
};
const TileTimes* tile_times(const Config& c) {
  static const std::array<const TileTimes*, kNumConfigs> of = [] {
    std::array<const TileTimes*, kNumConfigs> r{};
    for (const TileTimes& t : kTileTimes)
      if (const int i = find_config(t.name); i >= 0) r[(size_t)i] = &t;
    return r;
  }();
  return of[(size_t)(&c - kConfigs)];
}

// What the bytes of A, B and C take (TB/s), and that together with the time of the work: near the larger of the two.
double with_memory(double work, const gemm_desc_t& d, int64_t N) {
  const SharedTimes& h = d.dtype_a == GEMM_F8E4M3 ? kShared8 : kShared16;
  const double M = (double)d.M, n = (double)N, K = (double)d.K;
  const double c = d.dtype_c == GEMM_F32 ? M * n * 4.0 / h.c32 : M * n * 2.0 / h.c16;
  const double memory = h.launch + (double)d.batch * ((M + n) * K * esize(d.dtype_a) / h.operands + c) / 1e6;
  return std::sqrt(std::cbrt(std::pow(work, 6) + std::pow(memory, 6)));
}

double tile_cost(const Config& c, const TileTimes& t, const gemm_desc_t& d, int64_t N, double tiles, int off_line) {
  const double at_once = 160 * 1024 / c.lds_bytes, area = (double)c.bm * c.bn / (128 * 128);
  const SharedTimes& h = d.dtype_a == GEMM_F8E4M3 ? kShared8 : kShared16;
  const double turns = tiles / (num_cus() * at_once), whole = std::floor(turns), part = turns - whole;
  // (of a batch: the kernels that give an XCD whole problems, where tiles divide by 8, find shared panels in its L2)
  const bool apart = d.batch > 1 && !((persists(c, d) || c.t1 > 0) && std::fmod(tiles, 8.0) == 0);
  const double turn = t.tile + t.slab * (double)((d.K + c.bk - 1) / c.bk) * (1.0 + h.off_line * off_line + (apart ? h.apart : 0.0)) +
                      (d.dtype_c == GEMM_F32 ? h.f32 * area * at_once : 0.0);
  return with_memory(h.launch + turn * (whole + (part > 0 ? t.part + (1.0 - t.part) * part : 0.0)), d, N);
}

// (64x64 tiles of any alignment with both operands K-contiguous keep two slabs on their way: 0.78 of the time of a slab, with at most
// a tile per CU; 7692x369x7149, three per CU, takes 143 us on 128x128 tiles and 153 on these.)
// The others, 16-bit rings of 32 columns and for operands of any alignment, are weighed by the time of a slab with one workgroup
// on a CU and with two (launch 2.7 us; each further round costs 2.4 us of prologue and epilogue that nothing overlaps: 512x512x128,
// 64 problems, 64x64 tiles: 27 us).  An operand whose rows do not start on 128-byte lines costs a ring 0.35 on top: every piece of
// 128 bytes touches two lines (384x4104x4104: 43 us, 384x4096x4096: 24 us).  In a batch, the slices of split-K among them, a slab
// takes a quarter more: 1500 split-K products are then 0.7 % from the better of two estimates' choices, 3.3 % without.
double mfma_cost(const Config& c, const gemm_desc_t& d, int64_t N) {
  const int64_t M = d.M, K = d.K, batch = d.batch;
  const int e = esize(d.dtype_a);
  const double tiles = (double)((M + c.bm - 1) / c.bm) * (double)((N + c.bn - 1) / c.bn) * (double)batch;
  const double cus = num_cus();
  const int off_line = ((d.lda * e) % 128 != 0) + ((d.ldb * e) % 128 != 0);
  if (const TileTimes* t = tile_times(c)) return tile_cost(c, *t, d, N, tiles, off_line);
  const double slabs = (double)((K + c.bk - 1) / c.bk);
  const double per_cu = (double)(int64_t)((tiles + cus - 1) / cus);
  const bool tiled = c.kind != KIND_MFMA_G, many = tiled && batch > 1;
  const bool two_ahead = c.kind == KIND_MFMA_G && c.bm == 64 && per_cu <= 1 && d.layout_a == GEMM_ROW_MAJOR && d.layout_b == GEMM_COL_MAJOR;
  const double pitch = two_ahead ? 0.78 : c.kind == KIND_MFMA_G ? 1.0 : 1.0 + 0.35 * off_line + (many ? 0.25 : 0.0);
  const double pairs = c.t2 > 0 ? (double)(int64_t)(per_cu / 2) : 0.0, singles = per_cu - 2 * pairs;
  const double work = 2.7 + (singles * c.t1 + pairs * c.t2) * slabs * pitch + (singles + pairs - 1) * 2.4 + (many ? 0.7 : 0.0);
  return tiled ? with_memory(work, d, N) : work;               // (those are weighed against tile_cost's)
}

// Where the built-in choice weighs the kernels whose waves split K, which take rows on 128-byte lines only (a slab's rows of 128 bytes
// touch two otherwise: 502x1838, K = 4224 5 % ahead of the ring kernel, 1034x210, K = 10824 9 to 25 % behind): at most a tile per CU, and a K long
// enough for the addition of the waves' sums.  Time over the better ring kernel's of the same tile, drawn products, operands from HBM / in the
// last-level cache: 32x32 tiles, three tile rows and more from K = 1216 0.89 to 1.00 / 0.76 to 0.96, fewer rows from K = 2368 0.91 to 1.02 / 0.72 to
// 0.99 (below: up to 1.05); 64x64 tiles, four rows and columns of tiles and more from K = 1408 0.87 to 1.04 / 0.82 to 1.06; with fewer rows, where HBM
// alone is the bound, up to 1.08.
bool weighs_ksplit(const Config& c, const gemm_desc_t& d) {
  const int64_t tm = (d.M + c.bm - 1) / c.bm, tn = (d.N + c.bn - 1) / c.bn;
  if (tm * tn > num_cus() || tm * tn * d.batch > num_cus()) return false;
  return c.bm == 64 ? tm >= 4 && tn >= 4 && d.K >= 1408 : d.K >= (tm >= 3 ? 1216 : 2368);
}

// (ksplit: may it be one of those?  Not the inner product of a split-K plan, whose slices are parts of K already.)
int best_mfma(const gemm_desc_t& d, double* cost_out, bool ksplit = true) {
  int best = -1;
  double best_cost = 0;
  for (int i = 0; i < kNumConfigs; ++i) {
    const Config& c = kConfigs[i];
    if ((c.kind != KIND_MFMA && c.kind != KIND_MFMA_T && c.kind != KIND_MFMA_G) || !applicable(c, d)) continue;
    if (c.persist == 4 && !(ksplit && weighs_ksplit(c, d))) continue;
    if (c.persist == 2 && !persists(c, d)) continue;           // (the same kernel as the entry with one tile per workgroup)
    const double cost = mfma_cost(c, d, d.N);
    if (best < 0 || cost < best_cost) { best = i; best_cost = cost; }
  }
  if (cost_out) *cost_out = best_cost;
  return best;
}

// Wave quantisation: when the 256x256 tiles of a problem fill some whole rounds of the 256
// CUs and then a partial one, give the whole rounds to the big tile and the remaining
// columns to whatever tile shape suits them best (usually 128x128, two per CU).  Returns
// the number of leading columns for the first launch, or 0 for "do not split".
int64_t split_columns(const gemm_desc_t& d, int big, double single_cost) {
  if (big < 0 || d.batch != 1) return 0;
  const Config& c = kConfigs[big];
  if (c.bm != 256 || c.bn != 256) return 0;
  const int64_t tiles_m = (d.M + c.bm - 1) / c.bm, tiles_n = (d.N + c.bn - 1) / c.bn;
  if (tiles_m > num_cus() || num_cus() % tiles_m != 0) return 0;
  const int64_t cols_per_round = num_cus() / tiles_m;
  const int64_t cols_big = tiles_n / cols_per_round * cols_per_round;
  if (cols_big == 0 || cols_big == tiles_n) return 0;
  const int64_t n_first = cols_big * c.bn;
  gemm_desc_t rest = d;
  rest.N = d.N - n_first;
  double rest_cost = 0;
  if (best_mfma(rest, &rest_cost) < 0) return 0;
  // What the second launch takes beyond the two estimates, which count a launch each and no overlap.  Where the line lies, over drawn
  // products that can take two launches (1 to 6 rounds, K from 64 to 8192; taken, more than 2 % faster so, more than 2 % slower):
  // 16-bit results 1671: 307, 179, 24 with 1 us; 611, 211, 201 with -2; 218, 144, 14 with 3.  fp32 results 971: 408, 191, 107 with -2
  // (mean -1.4 %); 302, 168, 46 with -1; 135, 105, 9 with 2 (-1.1 %); 1024x17416x136 takes 29.0 us, 31.7 in one.  fp8, 2295
  // (mean -1.2 %): 598, 339, 72 with 2; 883, 401, 189 with 0; 266, 202, 18 with 7.
  const double launch = d.dtype_a == GEMM_F8E4M3 ? 2.0 : d.dtype_c == GEMM_F32 ? -2.0 : 0.5;
  return mfma_cost(c, d, n_first) + rest_cost + launch < single_cost ? n_first : 0;
}

// The choice among the general kernels (fp32 operands, or layouts / leading dimensions / pointers the tiled
// kernels do not take).
int choose_general(const gemm_desc_t& d) {
  //   * fp32, at most four 16x16 tiles per CU: 16x16 tiles with K split over the waves of a workgroup
  //     (256^3: 5 us against 11 us for the next choice; 512^3: 11 to 12 against 19 us);
  //   * fp32, up to eight 16x16 tiles per CU: those or 64x64 tiles, by an estimate;
  //   * very few 32x32 tiles (16-bit operands in layouts the tiled kernels do not take): the vector-ALU
  //     kernel with 32x32 tiles and the long K step;
  //   * fp32 in float4 groups: the fp32-MFMA kernels with slabs straight to LDS, 128x128 tiles from four
  //     tiles per CU on (4096^3: 0.94 to 0.96 ms = 143 to 147 TFLOP/s, 64x64 tiles 1.03 to 1.05, the general kernel 1.47),
  //     64x64 tiles below (3000^3: 444 us, 2048^3: 143 to 149, 1024^3: 24; general kernel 658 / 213 / 53 us);
  //   * otherwise the general fp32-MFMA kernel: 64x64 tiles until there are four 128x128 tiles per CU.
  const double tiles32 = (double)((d.M + 31) / 32) * (double)((d.N + 31) / 32) * d.batch;
  const double tiles128 = (double)((d.M + 127) / 128) * (double)((d.N + 127) / 128) * d.batch;
  if (tiles32 <= 1.0 * num_cus()) {             // (tiles32 = a quarter of the 16x16 tiles)
    const int i = find_config("f32small_16x16x256");
    if (i >= 0 && applicable(kConfigs[i], d)) return i;
  }
  if (tiles32 <= 2.0 * num_cus()) {
    // fp32: 16x16 tiles or 64x64 ones.  K up to 64: 64x64, within 2 % of the fastest kernel however many there are, 16x16 ones up to three
    // times that.  Beyond, microseconds fitted to half of 4326 drawn products with 257 to 512 32x32 tiles (all layouts, batches, K to
    // 4000; rms 15 and 8 %): the choice is 1.5 % from the better kernel on the other half (an estimate that looked at B's layout only and
    // took every problem for one 64x64 tile per CU: 4.8 %).  1079x467x529: 21.8 on 64x64 tiles, 33 on 16x16 ones, 29 on the vector-ALU
    // kernel; 2456x110x2930 117, 81 and 129; 512 problems of 32x32x2000 72, 106 and 94; 294 of 10x7x26, A column-major, 6.8, 8.4 and 6.7.
    const int small = find_config("f32small_16x16x256"), aligned = find_config("f32mfma_64x64x32");
    if (d.dtype_a == GEMM_F32 && f32_takes_any(d, 64) && small >= 0 && applicable(kConfigs[small], d)) {
      const bool pieces = applicable(kConfigs[aligned], d), b_row = d.layout_b == GEMM_ROW_MAJOR;
      const double K = (double)d.K, turns = (double)((d.M + 15) / 16) * (double)((d.N + 15) / 16) * d.batch / num_cus();
      const double tiles64 = (double)((d.M + 63) / 64) * (double)((d.N + 63) / 64) * d.batch / num_cus();
      const double k16 = d.layout_a == GEMM_ROW_MAJOR ? (b_row ? 0.0049 : 0.0038) : (b_row ? 0.0053 : 0.0044);
      // A few rows or columns and 64x64 tiles that take pieces: those load one piece of a row many times, and 16x16 ones read lines that
      // they share.  Both operands K-contiguous: 16x16 tiles (0.65 to 0.85 of the other's time at K > 256, 0.9 to 1.1 at K of 65 to 160);
      // else less than they are charged otherwise, least if the wide operand is K-contiguous.  By this rule 22050 drawn products (up to 16 rows or
      // columns, K from 65) are 1.0 % from the better kernel, from 2.2 % with the factor 0.84 of the other layouts, and 3.8 % of them
      // more than 10 % (8.1): 139 of 96x2x408 9.9 on 16x16 tiles, 20.1 on 64x64 ones; 70 of 4x208x2132, strided, 45 and 79.
      const bool few = d.M <= 16 || d.N <= 16, a_k = d.layout_a == GEMM_ROW_MAJOR;
      if (few && pieces && a_k && !b_row && d.K > 64) return small;
      const double narrow = few && pieces ? ((d.M < d.N ? !b_row : a_k) ? 0.7 : 0.8) : few && d.K > 256 ? 0.84 : 1.0;
      const double t16 = (few && pieces ? 5.85 : 4.85) + narrow * std::hypot(turns * (0.82 + k16 * K), 0.37e-6 * 4.0 * (double)(d.M + d.N) * K * d.batch);   // (operands at 2.7 TB/s)
      const double t64 = pieces ? 6.19 + (1.0 + 0.8 * fmax(0.0, tiles64 - 1.0)) * (0.0207 * K - 0.99)
                                : 5.11 + (1.0 + 0.8 * fmax(0.0, tiles64 - 1.0)) * ((b_row ? 0.0322 : 0.0253) * K - 0.09);
      return d.K > 64 && t16 < t64 ? small : pieces ? aligned : find_config("general_mfma32_64x64x16");
    }
    return find_config("simt_32x32x64");
  }
  {                                             // fp32 in float4 groups: 128x128 tiles from four per CU on
    const int i = find_config(tiles128 >= 4.0 * num_cus() ? "f32mfma_128x128x32" : "f32mfma_64x64x32");
    if (i >= 0 && applicable(kConfigs[i], d)) return i;
  }
  // fp32 of any alignment, many tiles: f32_any_kernel, whose registers and LDS allow five workgroups on a CU, is 1.02 to 1.24 behind the
  // general kernel with a few rows or columns and a K of one of that one's steps, 1.0 to 1.1 with K > 64 and more than five tiles per CU, and
  // 1.1 to 1.3 with K <= 8 and C column-major (20000 drawn products; fewer tiles, a K of one or two slabs: up to 0.8 ahead).
  const double tiles64 = (double)((d.M + 63) / 64) * (double)((d.N + 63) / 64) * d.batch / num_cus();
  const int64_t narrow = d.M < d.N ? d.M : d.N;
  if (d.dtype_a == GEMM_F32 && ((narrow <= 32 && ((d.K <= 16 && tiles64 > 3) || (d.K > 64 && tiles64 > 5))) ||
                                (d.K <= 8 && d.layout_c == GEMM_COL_MAJOR && tiles64 > 4)))
    return find_config("f32general_64x64x16");
  // (128x128 tiles of an fp32 problem that fills half of one: 2054x40x1, 227 problems, 120 us)
  const bool wide = d.dtype_a != GEMM_F32 || narrow > 64;
  return find_config(wide && tiles128 >= 4.0 * num_cus() ? "general_mfma32_128x128x16" : "general_mfma32_64x64x16");
}

// The choice for 16-bit operands of any alignment with K <= 64, where writing C and the fixed cost of a tile are most of the
// time and the general kernel, whose K step is 16, can win: microseconds of each kernel, fitted to 2081 drawn problems with
// K up to 256 (rms 13 to 19 %); fill: how much of its tiles a problem covers.  Of 4900 others with K <= 64, 250 were more than
// 5 % slower than on the general kernels with the any-alignment tiles throughout, 100 of them by more than 20 % (127 problems
// of 613x21x15: 19.2 against 7.8 us; 2319x879x9 with column-major C: 10.4 against 7.3); by this rule 90 and 24, and the mean
// is 1.4 % better.
int choose_short_k(const gemm_desc_t& d, int best) {
  const double cus = num_cus();
  const bool col = d.layout_c == GEMM_COL_MAJOR;             // (the general kernel writes 128 bytes of a column at a time)
  auto estimate = [&](int tile, int step, double fixed, double per_tile, double per_step, double per_fill) {
    const double tiles = (double)((d.M + tile - 1) / tile) * (double)((d.N + tile - 1) / tile) * d.batch;
    const double fill = (double)d.M * (double)d.N * d.batch / (tiles * tile * tile);
    return fixed + fmax(1.0, tiles / cus) * (per_tile + per_step * (double)((d.K + step - 1) / step) + per_fill * fill);
  };
  const double general = estimate(64, 16, 4.3, -0.7, 0.92, 2.3) * (col ? 0.7 : 1.1);
  const double g64 = estimate(64, 64, 4.7, 0.5, 0.48, 1.5) * (col ? 0.9 : 1.0);
  const double g128 = estimate(128, 64, 2.5, 3.4, 0.97, 4.9) * (col ? 0.95 : 1.0);
  const int i = find_config(general <= fmin(g64, g128) ? "general_mfma32_64x64x16"
                            : g64 <= g128 ? "mfma16g_64x64_k1_w2x2" : "mfma16g_128x128_k1_w2x4");
  return i >= 0 && applicable(kConfigs[i], d) ? i : best;
}

// Built-in choice.  MFMA tile: cheapest under a small cost model (wave quantisation over
// the 256 CUs, measured efficiency per tile shape); first entry of the table on ties.
int choose(const gemm_desc_t& d) {
  // skinny: up to 4 rows of x on the vector ALUs (smallest padded M that fits, first
  // such entry of the table), up to 16 on the matrix cores
  if (d.M > 1 && d.M <= 16) {
    // W through wave-private LDS slabs, 16x16x32 MFMA, two slabs requested ahead per wave, x in registers or its fragments
    // straight from L2 (M = 16: 24.3 us at N = K = 8192, 73.5 at N = 28672; M = 4: 23.0 us at N = 8192, where the vector-ALU
    // kernel below needs 26)
    const int rows = find_config("skinnydirect_d2_b512_w4_rows"), i = find_config("skinnydirect_d2_b512_w4");
    if (applicable(kConfigs[rows], d) && skinny_takes_rows(d)) return rows;
    if (applicable(kConfigs[i], d)) return i;
  }
  if (d.M <= 4) {
    // two waves per SIMD (8 per workgroup, one workgroup per CU) stream faster than one; for
    // long weight matrices two such workgroups per CU are a little better still (M = 1)
    const char* name = d.M == 1 ? (d.N >= 16384 ? "skinny_m1_w8_g2" : "skinny_m1_w8_g1")
                       : d.M == 2 ? "skinny_m2_w8_g1" : "skinny_m4_w8_g1";
    const int i = find_config(name);
    if (i >= 0 && applicable(kConfigs[i], d)) return i;
    int best = -1;
    for (int q = 0; q < kNumConfigs; ++q)
      if (kConfigs[q].kind == KIND_SKINNY && applicable(kConfigs[q], d) &&
          (best < 0 || kConfigs[q].bm < kConfigs[best].bm))
        best = q;
    if (best >= 0) return best;
  }
  const int best = best_mfma(d, nullptr);
  // operands of any alignment: up to 2^24 multiply-adds with a short K stay on the vector-ALU kernel (256x256x100: 6.5 us
  // on either; 25x933x453: 28 us there, 10 us on the matrix cores)
  if (best >= 0 && kConfigs[best].kind == KIND_MFMA_G && d.K <= 256 && (double)d.M * d.N * d.K * d.batch <= 16777216.0)
    return choose_general(d);
  if (best >= 0 && kConfigs[best].kind == KIND_MFMA_G && d.K <= 64) return choose_short_k(d, best);
  if (best >= 0) return best;
  return choose_general(d);
}

int fill_launch_shape(gemm_plan& pl) {
  const gemm_desc_t& d = pl.d;
  const Config& c = *pl.cfg;
  pl.block = dim3(c.threads, 1, 1);
  pl.xcd_remap = 0;
  if (c.kind == KIND_SIMT || c.kind == KIND_F32_VEC) {
    const int64_t gx = (d.N + c.bn - 1) / c.bn, gy = (d.M + c.bm - 1) / c.bm;
    if (gy > 65535) return GEMM_ERR_BAD_DIM;   // grid.y / grid.z limits
    pl.grid = dim3((unsigned)gx, (unsigned)gy, (unsigned)d.batch);
  } else if (c.kind == KIND_MFMA || c.kind == KIND_MFMA_T || c.kind == KIND_MFMA_G) {
    const int64_t tm = (d.M + c.bm - 1) / c.bm, tn = (d.N + c.bn - 1) / c.bn;
    int64_t wgs = tm * tn;
    const bool persist = persists(c, d);
    if (persist) {
      // as many workgroups as run at once; workgroup b takes tiles b, b + wgs, ... of all problems of the batch
      const int64_t at_once = (int64_t)num_cus() * (160 * 1024 / c.lds_bytes);
      wgs *= d.batch;
      if (wgs > at_once) wgs = at_once;
      pl.grid = dim3((unsigned)wgs, 1, 1);
    } else {
      pl.grid = dim3((unsigned)wgs, (unsigned)d.batch, 1);
    }
    pl.xcd_remap = d.batch == 1 || (tm * tn) % 8 == 0 ? 1 : 0;
    if (d.batch == 1 && dealt_one_by_one(tm, tn, c.bm * c.bn, d.K * esize(d.dtype_a), c.kind == KIND_MFMA_G && d.layout_b == GEMM_ROW_MAJOR))
      pl.xcd_remap = 0;
    // a batch, one tile per workgroup, on the kernels with a deeper ring: whole problems per XCD as well (512x512x2048,
    // 16 problems: 33 us with a problem's tiles spread over the XCDs)
    if (c.t1 > 0 && d.batch > 1 && (tm * tn * d.batch) % 8 == 0) {
      pl.grid = dim3((unsigned)(tm * tn * d.batch), 1, 1);
      pl.xcd_remap = 3;
    }
    // a batch on persistent workgroups: whole problems per XCD (their tiles share panels)
    if (persist && d.batch > 1 && (tm * tn * d.batch) % 8 == 0 && wgs % 8 == 0) pl.xcd_remap = 2;
  } else if (c.persist == 3) {
    // as many workgroups as share the panels evenly, at most one per CU (896 panels: 224; 14336x8192 39.9 us with 256, 39.1 so)
    const int64_t panels = (d.N + c.bn - 1) / c.bn, turns = (panels + num_cus() - 1) / num_cus();
    pl.grid = dim3((unsigned)((panels + turns - 1) / turns), 1, 1);
  } else if (c.kind == KIND_SKINNY_PANEL) {
    pl.grid = dim3((unsigned)((d.N + c.bn - 1) / c.bn), (unsigned)d.batch, 1);
  } else {
    // One row of W per wave at a time, rows dealt round-robin: bn workgroups per CU,
    // more only if a wave would otherwise own more rows than the kernel has slots for.
    const int waves = c.threads / 64;
    int64_t wgs = (d.N + waves - 1) / waves;                       // one row per wave
    const int64_t want = (int64_t)num_cus() * c.bn;
    if (wgs > want) wgs = want;
    const int64_t need = (d.N + (int64_t)waves * kSkinnyMaxRows - 1) / ((int64_t)waves * kSkinnyMaxRows);
    if (wgs < need) wgs = need;
    pl.grid = dim3((unsigned)wgs, (unsigned)d.batch, 1);
  }
  return GEMM_OK;
}

// gfx950 check, once per device.
}  // namespace

// ---- C ABI -------------------------------------------------------------------------------

extern "C" {

// GEMM_LOG=1 in the environment: one line on stderr per plan, saying which kernel and tile it got.
static bool log_enabled() {
  static const bool on = [] {
    const char* e = std::getenv("GEMM_LOG");
    return e && e[0] && std::strcmp(e, "0") != 0;
  }();
  return on;
}

int gemm_config_count(void) { return kNumConfigs; }

const char* gemm_config_name(int config) {
  return (config >= 0 && config < kNumConfigs) ? kConfigs[config].name : nullptr;
}

// Plan for an already resolved descriptor.  allow_two_launches: the built-in choice may
// plan a second launch against wave quantisation.
static int create_resolved(const gemm_desc_t& d, int config, bool allow_two_launches, gemm_plan_t** out_plan) {
  if (config < -1 || config >= kNumConfigs) return GEMM_ERR_BAD_CONFIG;
  const bool auto_choice = config == -1;
  if (config == -1) config = choose(d);
  if (config < 0) return GEMM_ERR_UNSUPPORTED;
  if (!applicable(kConfigs[config], d)) return auto_choice ? GEMM_ERR_UNSUPPORTED : GEMM_ERR_BAD_CONFIG;
  gemm_plan* pl = new (std::nothrow) gemm_plan;
  if (!pl) return GEMM_ERR_NULL;
  pl->d = d;
  pl->cfg = &kConfigs[config];
  pl->cfg_index = config;
  pl->tail = nullptr;
  pl->tail_off_b = pl->tail_off_c = pl->tail_off_bias = 0;
  pl->fallback = nullptr;
  pl->splits = 0;
  pl->inner = nullptr;
  pl->d_user = d;
  pl->c_cached = 0;
  pl->built_in = auto_choice && allow_two_launches;   // (second launches and split-K inner plans are parts, not plans)
  pl->tune_state = 0;
  pl->tuned = nullptr;
  const Kind kind = kConfigs[config].kind;
  if (kind == KIND_MFMA_T) {
    // pointers need element alignment only, as for every problem these layouts were ever planned for
    const int rc = create_resolved(d, choose_general(d), false, &pl->fallback);
    if (rc != GEMM_OK) { gemm_destroy(pl); return rc; }
  }
  if (auto_choice && allow_two_launches && (kind == KIND_MFMA || kind == KIND_MFMA_T)) {
    double single_cost = 0;
    best_mfma(d, &single_cost);
    int big = -1;                                   // the first 256x256 shape of the table
    for (int i = 0; i < kNumConfigs && big < 0; ++i)
      if (kConfigs[i].kind == kind && kConfigs[i].bm == 256 && kConfigs[i].bn == 256 && applicable(kConfigs[i], d) &&
          !(kConfigs[i].persist == 2 && !persists(kConfigs[i], d)))
        big = i;
    const int64_t n_first = split_columns(d, big, single_cost);
    if (n_first > 0) {
      config = big;
      pl->cfg = &kConfigs[config];
      pl->cfg_index = config;
      // second launch: columns n_first .. N-1 (rows of the N x K weight matrix or columns of a K x N one, columns of C)
      gemm_desc_t rest = d;
      rest.N = d.N - n_first;
      gemm_plan_t* tail = nullptr;
      if (create_resolved(rest, best_mfma(rest, nullptr), false, &tail) == GEMM_OK) {
        pl->tail = tail;
        pl->tail_off_b = d.layout_b == GEMM_COL_MAJOR ? n_first * d.ldb : n_first;
        pl->tail_off_c = n_first;
        pl->tail_off_bias = n_first;
        pl->d.N = n_first;
      }
    }
  }
  const int rc = fill_launch_shape(*pl);
  if (rc != GEMM_OK) { gemm_destroy(pl); return rc; }
  *out_plan = pl;
  if (allow_two_launches && log_enabled()) {     // (second launches and split-K inner plans are reported with their parent)
    char buf[512];
    gemm_plan_info(pl, buf, sizeof(buf));
    std::fprintf(stderr, "[mi355gemm] plan %lld x %lld x %lld batch %d dtype %d -> %d epilogue %d: %s\n", (long long)d.M,
                 (long long)d.N, (long long)d.K, (int)d.batch, (int)d.dtype_a, (int)d.dtype_c, (int)d.epilogue, buf);
  }
  return GEMM_OK;
}

int gemm_create_config(const gemm_desc_t* desc, int config, gemm_plan_t** out_plan) {
  if (out_plan) *out_plan = nullptr;
  if (!desc || !out_plan) return GEMM_ERR_NULL;
  gemm_desc_t d;
  const int rc = resolve(desc, &d);
  if (rc != GEMM_OK) return rc;
  return create_resolved(d, config, true, out_plan);
}

// The two-slab tiles as the number of slices weighs them: rounds over the CUs * work per round / measured relative efficiency of the
// tile shape; a fixed per-tile cost (prologue latency, epilogue) is worth ~600 columns of K.
static double round_cost(const Config& c, const gemm_desc_t& d) {
  const int area = c.bm * c.bn;
  const double tiles = (double)((d.M + c.bm - 1) / c.bm) * (double)((d.N + c.bn - 1) / c.bn) * (double)d.batch;
  const double cus = num_cus();
  const int per_cu = area <= 128 * 128 ? 2 : 1;                 // workgroups that fit one CU's LDS
  double eff = area >= 256 * 256 ? 1.0 : (area >= 256 * 192 ? 0.88 : (area >= 256 * 128 ? 0.75 : 0.84));
  if (!std::strncmp(c.name, "mfma16", 6)) eff *= 1.10;
  const double rounds = (double)(int64_t)((tiles + cus * per_cu - 1) / (cus * per_cu));
  // workgroups that actually share a CU (a lone workgroup runs about per_cu times faster)
  const double sharing = tiles >= cus * per_cu ? per_cu : (tiles > cus ? tiles / cus : 1.0);
  return rounds * area * sharing / eff * ((double)d.K + 600.0) / 2.7e6;
}

// Slices of K for a split-K plan: the count (up to 64, K a multiple of 8 x slices, whole
// slabs per slice preferred) that minimises the round model of the two-slab tiles on the sliced product plus
// the traffic of the fp32 partials (written once, read once: priced at 2 TB/s).  512x512x32768 takes 31 / 25 / 38 / 40 us
// with 8 / 16 / 32 / 64 slices; the model picks 16.  (The count decides the workspace's size, whether the fixed scratch buffer
// holds it and how long the fp32 sums are, so it must not move when the choice of kernels is refitted: neither the four-slab
// kernels' model, which would take fewer slices and add more terms in each, nor tiles of 192 or 224 rows, nor the short-K
// terms of the estimate above take part.)
static int choose_splits(const gemm_desc_t& d) {
  int best = 1;
  double best_cost = 0;
  for (int pass = 0; pass < 2 && best_cost == 0; ++pass) {
    const int64_t epc = 16 / esize(d.dtype_a);
    const int64_t unit = pass == 0 ? 8 * epc : epc;          // whole slabs, else whole 16-byte pieces
    for (int64_t s = 1; s <= 64; ++s) {
      if (d.K % (s * unit) != 0) continue;
      gemm_desc_t in = d;
      in.K = d.K / s;
      in.batch = (int32_t)s;
      in.stride_a = in.stride_b = in.K;
      double cost = 0;
      for (int i = 0; i < kNumConfigs; ++i) {
        const Config& c = kConfigs[i];
        if (c.kind != KIND_MFMA || c.t1 > 0 || c.bm % 128 != 0 || !applicable(c, in)) continue;
        const double t = round_cost(c, in);
        if (cost == 0 || t < cost) cost = t;
      }
      if (cost == 0) continue;
      cost += 2.0 * (double)s * (double)d.M * (double)d.N * 4.0 / 2.0e6;
      if (best_cost == 0 || cost < best_cost) { best = (int)s; best_cost = cost; }
    }
  }
  return best;
}

int gemm_create_splitk(const gemm_desc_t* desc, int splits, gemm_plan_t** out_plan) {
  if (out_plan) *out_plan = nullptr;
  if (!desc || !out_plan) return GEMM_ERR_NULL;
  gemm_desc_t d;
  int rc = resolve(desc, &d);
  if (rc != GEMM_OK) return rc;
  if (splits < 0 || splits > 1024) return GEMM_ERR_BAD_DIM;
  if (d.batch != 1 || d.dtype_a == GEMM_F32) return GEMM_ERR_UNSUPPORTED;
  if (d.layout_a != GEMM_ROW_MAJOR || d.layout_b != GEMM_COL_MAJOR) return GEMM_ERR_UNSUPPORTED;
  if (splits == 0) splits = choose_splits(d);
  if (d.K % ((int64_t)splits * (16 / esize(d.dtype_a))) != 0) return GEMM_ERR_UNSUPPORTED;
  if ((double)splits * (double)d.M * (double)d.N * 4.0 >= 9.0e18) return GEMM_ERR_BAD_DIM;
  // the K slices as the batches of a product into packed fp32 partials, no epilogue
  gemm_desc_t in = d;
  in.K = d.K / splits;
  in.batch = splits;
  in.stride_a = in.K;                 // slice s of A starts K/splits columns further on
  in.stride_b = in.K;
  in.dtype_c = GEMM_F32;
  in.layout_c = GEMM_ROW_MAJOR;
  in.ldc = d.N;
  in.stride_c = d.M * d.N;
  in.epilogue = GEMM_EPI_NONE;
  in.stride_bias = 0;
  in.scale = 1.0f;
  // What split-K takes is what the K-contiguous kernels with two slabs take (best_mfma alone would also offer the
  // any-alignment kernels for leading dimensions that are not whole 16-byte pieces).
  bool taken = false;
  for (int i = 0; i < kNumConfigs && !taken; ++i) taken = kConfigs[i].kind == KIND_MFMA && kConfigs[i].t1 == 0 && applicable(kConfigs[i], in);
  if (!taken) return GEMM_ERR_UNSUPPORTED;
  const int inner_cfg = best_mfma(in, nullptr, false);
  if (inner_cfg < 0) return GEMM_ERR_UNSUPPORTED;
  gemm_plan_t* inner = nullptr;
  rc = create_resolved(in, inner_cfg, false, &inner);
  if (rc != GEMM_OK) return rc;
  inner->c_cached = 1;                // the reduction kernel reads the partials next
  if (inner->tail) inner->tail->c_cached = 1;
  gemm_plan* pl = new (std::nothrow) gemm_plan(*inner);
  if (!pl) { gemm_destroy(inner); return GEMM_ERR_NULL; }
  pl->d = d;
  pl->d_user = d;
  pl->built_in = 0;
  pl->splits = splits;
  pl->inner = inner;
  *out_plan = pl;
  return GEMM_OK;
}

size_t gemm_workspace_bytes(const gemm_plan_t* plan) {
  if (!plan || !plan->inner) return 0;
  return (size_t)plan->splits * (size_t)plan->d.M * (size_t)plan->d.N * 4;
}

int gemm_run_workspace(const gemm_plan_t* plan, const void* A, const void* B, void* C,
                       const void* bias, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!plan) return GEMM_ERR_NULL;
  if (!plan->inner) return gemm_run(plan, A, B, C, bias, hip_stream);
  if (!A || !B || !C) return GEMM_ERR_NULL;
  const gemm_desc_t& d = plan->d;
  if (epilogue_has_bias(d.epilogue) != (bias != nullptr)) return GEMM_ERR_NULL;
  if (!workspace || workspace_bytes < gemm_workspace_bytes(plan) || ((uintptr_t)workspace & 15))
    return GEMM_ERR_WORKSPACE;
  if (((uintptr_t)C & ((uintptr_t)esize(d.dtype_c) - 1)) || ((uintptr_t)bias & 3)) return GEMM_ERR_MISALIGNED;
  int rc = gemm_run(plan->inner, A, B, workspace, nullptr, hip_stream);
  if (rc != GEMM_OK) return rc;
  SplitKReduceArgs r;
  r.ws = (const float*)workspace; r.C = C; r.bias = (const float*)bias;
  r.M = d.M; r.N = d.N;
  r.c_si = d.layout_c == GEMM_ROW_MAJOR ? d.ldc : 1;
  r.c_sj = d.layout_c == GEMM_ROW_MAJOR ? 1 : d.ldc;
  r.splits = plan->splits;
  r.has_bias = epilogue_has_bias(d.epilogue);
  r.act = epilogue_activation(d.epilogue);
  r.scale = d.scale;
  const int64_t quads = d.M * ((d.N + 3) / 4);
  const int64_t blocks = (quads + 255) / 256;
  if (blocks >= ((int64_t)1 << 31)) return GEMM_ERR_BAD_DIM;
  hipStream_t s = (hipStream_t)hip_stream;
  switch (d.dtype_c) {
    case GEMM_F32: splitk_reduce_kernel<float><<<(unsigned)blocks, 256, 0, s>>>(r); break;
    case GEMM_BF16: splitk_reduce_kernel<bf16_t><<<(unsigned)blocks, 256, 0, s>>>(r); break;
    default: splitk_reduce_kernel<f16_t><<<(unsigned)blocks, 256, 0, s>>>(r); break;
  }
  return hipGetLastError() == hipSuccess ? GEMM_OK : GEMM_ERR_LAUNCH;
}

// ---- the fixed scratch buffer -----------------------------------------------------------------
// Device memory inside the code object: each GPU the library is loaded on has its own copy at
// its own address.  In host code the array's name is only a handle for hipGetSymbolAddress;
// the address it returns (per device, looked up once with that device current) is what kernels
// and launches are given.
static __device__ __align__(256) unsigned char g_fixed_scratch[GEMM_FIXED_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of the buffer, or nullptr.
void* fixed_scratch_of_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return nullptr; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_fixed_scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

int gemm_run_fixed_scratch(const gemm_plan_t* plan, const void* A, const void* B, void* C,
                           const void* bias, void* hip_stream) {
  if (!plan) return GEMM_ERR_NULL;
  if (!plan->inner) return gemm_run(plan, A, B, C, bias, hip_stream);
  const size_t need = gemm_workspace_bytes(plan);
  if (need > GEMM_FIXED_SCRATCH_BYTES) return GEMM_ERR_FIXED_SCRATCH;
  int rc = check_device_gfx950();
  if (rc != GEMM_OK) return rc;
  void* ws = fixed_scratch_of_current_device();
  if (!ws) return GEMM_ERR_LAUNCH;
  return gemm_run_workspace(plan, A, B, C, bias, ws, GEMM_FIXED_SCRATCH_BYTES, hip_stream);
}

int gemm_create(const gemm_desc_t* desc, gemm_plan_t** out_plan) {
  return gemm_create_config(desc, -1, out_plan);
}

// The launches of one plan, arguments checked; no tuning logic.
static int run_plan(const gemm_plan_t* plan, const void* A, const void* B, void* C, const void* bias,
                    void* hip_stream) {
  if (!plan || !A || !B || !C) return GEMM_ERR_NULL;
  if (plan->inner) return GEMM_ERR_WORKSPACE;
  if (plan->fallback && (((uintptr_t)A | (uintptr_t)B) & 15)) return run_plan(plan->fallback, A, B, C, bias, hip_stream);
  const gemm_desc_t& d = plan->d;
  if (epilogue_has_bias(d.epilogue) != (bias != nullptr)) return GEMM_ERR_NULL;
  // The tiled 16-bit kernels move 16-byte pieces; the general kernel only needs
  // element alignment.
  const Kind kind = plan->cfg->kind;
  const uintptr_t in_mask = kind == KIND_SIMT || kind == KIND_F32_VEC || kind == KIND_MFMA_G ? (uintptr_t)esize(d.dtype_a) - 1 : 15;
  if (((uintptr_t)A & in_mask) || ((uintptr_t)B & in_mask) ||
      ((uintptr_t)C & ((uintptr_t)esize(d.dtype_c) - 1)) || ((uintptr_t)bias & 3))
    return GEMM_ERR_MISALIGNED;
  int rc = check_device_gfx950();
  if (rc != GEMM_OK) return rc;
  hipError_t e = plan->cfg->launch[d.dtype_a](*plan, A, B, C, bias, (hipStream_t)hip_stream);
  if (e != hipSuccess) return GEMM_ERR_LAUNCH;
  if (plan->tail) {
    const gemm_plan* t = plan->tail;
    const char* B2 = (const char*)B + plan->tail_off_b * esize(d.dtype_b);
    char* C2 = (char*)C + plan->tail_off_c * esize(d.dtype_c);
    const float* bias2 = bias ? (const float*)bias + plan->tail_off_bias : nullptr;
    e = t->cfg->launch[d.dtype_a](*t, A, B2, C2, bias2, (hipStream_t)hip_stream);
    if (e != hipSuccess) return GEMM_ERR_LAUNCH;
  }
  return GEMM_OK;
}

// Mean microseconds per launch of one plan under the paper's timing protocol (App.
// "Benchmarking kernel runtime"): a few initial trials size the loops, a warm-up of at least
// min_seconds and 10 launches, then inner loops of >= min(0.01 s, min_seconds) between two
// event synchronisations until at least min_seconds and 10 launches have been measured.
static int time_plan(const gemm_plan_t* pl, const void* A, const void* B, void* C, const void* bias,
                     void* hip_stream, hipEvent_t e0, hipEvent_t e1, double min_seconds, double* us) {
  hipStream_t stream = (hipStream_t)hip_stream;
  int status = GEMM_OK;
  // n launches between two events; returns elapsed seconds (< 0 on failure)
  auto timed = [&](long n) -> double {
    if (hipEventRecord(e0, stream) != hipSuccess) return -1.0;
    for (long i = 0; i < n; ++i) {
      int r = run_plan(pl, A, B, C, bias, hip_stream);
      if (r != GEMM_OK) { status = r; return -1.0; }
    }
    if (hipEventRecord(e1, stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) return -1.0;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) return -1.0;
    return (double)ms * 1e-3;
  };
  auto failed = [&]() { return status != GEMM_OK ? status : GEMM_ERR_LAUNCH; };
  const double inner_s = min_seconds < 0.01 ? min_seconds : 0.01;
  double t = timed(3);                                   // initial trials: rough runtime
  if (t < 0) return failed();
  const double per = t / 3 > 1e-7 ? t / 3 : 1e-7;
  const long inner = (long)(inner_s / per) + 1;
  long warm = (long)(min_seconds / per) + 1;             // warm-up: at least min_seconds and 10 launches
  if (warm < 10) warm = 10;
  if (timed(warm) < 0) return failed();
  double total = 0.0;
  long launches = 0;
  while (total < min_seconds || launches < 10) {
    const double dt = timed(inner);
    if (dt < 0) return failed();
    total += dt;
    launches += inner;
  }
  *us = total / (double)launches * 1e6;
  return GEMM_OK;
}

int gemm_tune(const gemm_desc_t* desc, const void* A, const void* B, void* C, const void* bias,
              void* hip_stream, double min_seconds, int* best_config, float* us_per_config) {
  if (!desc || !A || !B || !C || !best_config) return GEMM_ERR_NULL;
  *best_config = -1;
  gemm_desc_t d;
  int rc = resolve(desc, &d);
  if (rc != GEMM_OK) return rc;
  if (!(min_seconds >= 0.0)) min_seconds = 0.0;
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) { (void)hipGetLastError(); return GEMM_ERR_LAUNCH; }
  if (hipEventCreate(&e1) != hipSuccess) { (void)hipGetLastError(); (void)hipEventDestroy(e0); return GEMM_ERR_LAUNCH; }
  double best_us = 0.0;
  int status = GEMM_OK;
  for (int i = 0; i < kNumConfigs && status == GEMM_OK; ++i) {
    if (us_per_config) us_per_config[i] = -1.0f;
    if (!applicable(kConfigs[i], d)) continue;
    gemm_plan_t* pl = nullptr;
    if (create_resolved(d, i, true, &pl) != GEMM_OK) continue;
    double us = 0.0;
    status = time_plan(pl, A, B, C, bias, hip_stream, e0, e1, min_seconds, &us);
    gemm_destroy(pl);
    if (status != GEMM_OK) break;
    if (us_per_config) us_per_config[i] = (float)us;
    if (*best_config < 0 || us < best_us) { *best_config = i; best_us = us; }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (status != GEMM_OK) { (void)hipGetLastError(); return status; }
  return *best_config >= 0 ? GEMM_OK : GEMM_ERR_UNSUPPORTED;
}

// ---- tuning mode --------------------------------------------------------------------------
// The paper's parameter optimisation (Sec. 3.4) as a switch: with it on, the first gemm_run of
// a problem times every applicable instantiation and the built-in plan on the caller's own
// buffers and remembers the winner per problem for the rest of the process.
namespace {

struct TuneKey {
  int64_t v[17];
  bool operator<(const TuneKey& o) const { return std::memcmp(v, o.v, sizeof(v)) < 0; }
};
TuneKey tune_key(const gemm_desc_t& d) {                 // everything but the epilogue's scalar
  TuneKey k;
  const int64_t f[17] = {d.M, d.N, d.K, d.batch, d.layout_a, d.layout_b, d.layout_c, d.dtype_a, d.dtype_b,
                         d.dtype_c, d.epilogue, d.lda, d.ldb, d.ldc, d.stride_a, d.stride_b, d.stride_c};
  std::memcpy(k.v, f, sizeof(f));
  return k;
}
std::mutex g_tune_mutex;
std::map<TuneKey, int> g_tune_cache;                     // problem -> fastest configuration, -1 = the built-in plan
std::atomic<int> g_autotune{-1};                         // -1: not yet read from the environment
constexpr double kAutotuneSeconds = 0.02;                // per configuration: warm-up and measurement each

bool autotune_on() {
  int v = g_autotune.load();
  if (v < 0) {
    const char* e = std::getenv("GEMM_TUNE");
    int from_env = (e && e[0] && std::strcmp(e, "0") != 0) ? 1 : 0;
    int expected = -1;
    g_autotune.compare_exchange_strong(expected, from_env);
    v = g_autotune.load();
  }
  return v == 1;
}

// Decide how `plan` runs from now on (tune_state 1: as it is; 2: through plan->tuned).
int autotune_plan(const gemm_plan_t* plan, const void* A, const void* B, void* C, const void* bias,
                  void* hip_stream) {
  gemm_plan_t* self = const_cast<gemm_plan_t*>(plan);    // only the two set-once tuning fields are written
  const gemm_desc_t& d = plan->d_user;
  std::lock_guard<std::mutex> lock(g_tune_mutex);         // one tuning run at a time; later callers find the entry
  if (__atomic_load_n(&self->tune_state, __ATOMIC_ACQUIRE) != 0) return GEMM_OK;
  int cfg = -1;
  const TuneKey key = tune_key(d);
  auto it = g_tune_cache.find(key);
  if (it != g_tune_cache.end()) {
    cfg = it->second;
  } else {
    int best = -1;
    std::vector<float> us(kNumConfigs, -1.0f);
    int rc = gemm_tune(&d, A, B, C, bias, hip_stream, kAutotuneSeconds, &best, us.data());
    if (rc != GEMM_OK) return rc;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) { (void)hipGetLastError(); return GEMM_ERR_LAUNCH; }
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipGetLastError(); (void)hipEventDestroy(e0); return GEMM_ERR_LAUNCH; }
    double own = 0.0;
    rc = time_plan(plan, A, B, C, bias, hip_stream, e0, e1, kAutotuneSeconds, &own);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != GEMM_OK) { (void)hipGetLastError(); return rc; }
    // a configuration replaces the built-in plan only for a clear win
    const bool same = best == plan->cfg_index && !plan->tail;
    cfg = (!same && (double)us[best] < 0.98 * own) ? best : -1;
    g_tune_cache[key] = cfg;
  }
  if (cfg >= 0 && !(cfg == plan->cfg_index && !plan->tail)) {
    gemm_plan_t* tp = nullptr;
    const int rc = create_resolved(d, cfg, true, &tp);
    if (rc != GEMM_OK) return rc;
    tp->built_in = 0;
    self->tuned = tp;
    __atomic_store_n(&self->tune_state, 2, __ATOMIC_RELEASE);
  } else {
    __atomic_store_n(&self->tune_state, 1, __ATOMIC_RELEASE);
  }
  return GEMM_OK;
}

}  // namespace

int gemm_set_autotune(int enabled) {
  const int before = autotune_on() ? 1 : 0;
  g_autotune.store(enabled ? 1 : 0);
  return before;
}

int gemm_autotune_entries(void) {
  std::lock_guard<std::mutex> lock(g_tune_mutex);
  return (int)g_tune_cache.size();
}

int gemm_autotune_clear(void) {
  std::lock_guard<std::mutex> lock(g_tune_mutex);
  g_tune_cache.clear();
  return GEMM_OK;
}

int gemm_run(const gemm_plan_t* plan, const void* A, const void* B, void* C, const void* bias,
             void* hip_stream) {
  if (plan && plan->built_in && !plan->inner && autotune_on()) {
    int state = __atomic_load_n(&plan->tune_state, __ATOMIC_ACQUIRE);
    if (state == 0) {
      // arguments are checked before anything is timed with them
      if (!A || !B || !C) return GEMM_ERR_NULL;
      if (epilogue_has_bias(plan->d.epilogue) != (bias != nullptr)) return GEMM_ERR_NULL;
      if (((uintptr_t)A & 15) || ((uintptr_t)B & 15) || ((uintptr_t)C & 15) || ((uintptr_t)bias & 3))
        return run_plan(plan, A, B, C, bias, hip_stream);   // (unusual alignment: no tuning, the plan's own checks decide)
      const int rc = autotune_plan(plan, A, B, C, bias, hip_stream);
      if (rc != GEMM_OK) return rc;
      state = __atomic_load_n(&plan->tune_state, __ATOMIC_ACQUIRE);
    }
    if (state == 2) return run_plan(plan->tuned, A, B, C, bias, hip_stream);
  }
  return run_plan(plan, A, B, C, bias, hip_stream);
}

int gemm_destroy(gemm_plan_t* plan) {
  if (plan) {
    if (plan->inner) {                 // a split-K plan is a copy of its inner plan's launch data
      gemm_destroy(plan->inner);
    } else {
      if (plan->tail) gemm_destroy(plan->tail);
      if (plan->fallback) gemm_destroy(plan->fallback);
      if (plan->built_in && plan->tuned) gemm_destroy(plan->tuned);
    }
  }
  delete plan;
  return GEMM_OK;
}

const char* gemm_status_string(int status) {
  switch (status) {
    case GEMM_OK: return "ok";
    case GEMM_ERR_NULL: return "null pointer (or bias does not match the epilogue)";
    case GEMM_ERR_BAD_DIM: return "bad dimension";
    case GEMM_ERR_BAD_LD: return "bad leading dimension or batch stride";
    case GEMM_ERR_UNSUPPORTED: return "unsupported dtype / layout / epilogue combination";
    case GEMM_ERR_MISALIGNED: return "misaligned pointer";
    case GEMM_ERR_NO_DEVICE: return "current device is not a gfx950 GPU";
    case GEMM_ERR_LAUNCH: return "kernel launch failed";
    case GEMM_ERR_BAD_ENUM: return "enum value out of range";
    case GEMM_ERR_BAD_CONFIG: return "tile configuration unknown or not applicable";
    case GEMM_ERR_BAD_SCALE: return "epilogue scale is not finite";
    case GEMM_ERR_WORKSPACE: return "plan needs a workspace (gemm_run_workspace), or the workspace is too small or misaligned";
    case GEMM_ERR_FIXED_SCRATCH: return "plan needs more workspace than the library's fixed scratch buffer of 32 MiB (use gemm_run_workspace)";
    default: return "unknown status";
  }
}

int gemm_plan_info(const gemm_plan_t* plan, char* buf, size_t n) {
  if (!plan || (!buf && n)) return GEMM_ERR_NULL;
  if (plan->built_in && __atomic_load_n(&plan->tune_state, __ATOMIC_ACQUIRE) == 2) {
    // timed in tuning mode and replaced: report what runs
    const int len = gemm_plan_info(plan->tuned, buf, n);
    if (len < 0) return len;
    const char* tag = " (tuned)";
    if (buf && (size_t)len < n) std::snprintf(buf + len, n - (size_t)len, "%s", tag);
    return len + (int)std::strlen(tag);
  }
  const Config& c = *plan->cfg;
  if (plan->inner) {
    const Runs r = plan_runs(*plan->inner);
    return std::snprintf(buf, n, "kernel=splitk_%d+%s tile=%dx%dx%d grid=%u,%u,%u block=%u lds=%d workspace=%zu",
                         plan->splits, c.name, c.bm, c.bn, r.bk, plan->grid.x, plan->grid.y, plan->grid.z,
                         plan->block.x, r.lds, gemm_workspace_bytes(plan));
  }
  const Runs r = plan_runs(*plan);
  char other[96] = "";
  if (plan->fallback) std::snprintf(other, sizeof(other), " unaligned A or B: kernel=%s", plan->fallback->cfg->name);
  if (plan->tail) {
    const Config& t = *plan->tail->cfg;
    return std::snprintf(buf, n, "kernel=%s tile=%dx%dx%d grid=%u,%u,%u block=%u lds=%d columns=0..%lld "
                         "+ kernel=%s grid=%u,%u,%u columns=%lld..%s", c.name, c.bm, c.bn, r.bk,
                         plan->grid.x, plan->grid.y, plan->grid.z, plan->block.x, r.lds,
                         (long long)plan->d.N - 1, t.name, plan->tail->grid.x, plan->tail->grid.y,
                         plan->tail->grid.z, (long long)plan->d.N, other);
  }
  return std::snprintf(buf, n, "kernel=%s tile=%dx%dx%d grid=%u,%u,%u block=%u lds=%d%s", c.name,
                       c.bm, c.bn, r.bk, plan->grid.x, plan->grid.y, plan->grid.z, plan->block.x, r.lds, other);
}

}  // extern "C"
