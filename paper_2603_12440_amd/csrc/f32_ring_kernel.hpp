// fp32 GEMM on the matrix cores with slabs of K in a ring (v_mfma_f32_32x32x2_f32: exact fp32 products, fp32
// accumulation), 64x64 or 128x128 tiles, for operands that can be moved in 16-byte pieces.
//
// f32_mfma_kernel.hpp stages its slabs through registers: every slab costs address arithmetic, LDS writes and a wait for
// loads that were requested one slab earlier, on the critical path of a wave that has one 32x32 tile to multiply.  Here
// the slabs go global -> LDS directly (NSTAGE - 1 of them on their way, one barrier each), as in ring_kernel.hpp.
// 64x64 tiles (three stages, three workgroups per CU) 2000x1500x1100 77.5 -> 58.2 us, 1024^3 41 -> 24; 128x128 tiles (two
// stages, two workgroups) 4096^3 1183 -> 962 us = 143 TFLOP/s.  Bound by the fp32 matrix pipes (157 TFLOP/s) in the large,
// by how evenly the tiles divide over the CUs and by one turn of barrier and LDS reads per slab in the small.
// LDS: K contiguous, 128-byte rows of 32 values, 16-byte chunk c of row r at slot c ^ swz16(r); K strided, 1 KB blocks
// of 8 values of K x 32 rows (block = 4 (row / 32) + k / 8), value k at 128-byte line (k ^ bit 2 of k) % 8 of its block,
// so that the two halves of a wave, which multiply k and k + 4, read different halves of the banks.
// An MFMA takes two columns of K, one from each half of the wave; which two is free as long as A and B agree: half h
// takes columns 8 j + 4 h + e (j, e = 0 .. 3), a 16-byte piece at a time where K is contiguous.
#pragma once

#include "mfma_kernel.hpp"
#include "mfma16_kernel.hpp"

namespace mi355gemm {

// Slabs in LDS for a tile of this height: three workgroups fit a CU with 64x64 tiles, two with 128x128.
constexpr int f32_ring_stages(int tile) { return tile == 64 ? 3 : 2; }

// MT: 32x32 tiles of a wave in each direction (tile 64 MT x 64 MT, 2 x 2 waves)
template <bool A_KF, bool B_KF, int MT, int NSTAGE>
__global__ __launch_bounds__(256) void f32_ring_kernel(MfmaArgs p, int64_t c_si, int64_t c_sj) {
  static_assert(NSTAGE == 2 || NSTAGE == 3, "at most one slab on its way behind the one waited for");
  constexpr int BM = 64 * MT, BN = 64 * MT, BK = 32;
  constexpr int A_BYTES = BM * 128, STAGE = 2 * A_BYTES, HALF = 2 * MT, LOADS = 2 * HALF;   // loads of A, and of both, per wave and slab
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NSTAGE * STAGE];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int fr = lane & 31, fh = lane >> 5;
  const int64_t batch = blockIdx.z;
  int tm, tn;
  tile_coords<false>(p, blockIdx.y * gridDim.x + blockIdx.x, p.tiles_m * p.tiles_n, tm, tn);
  const int r0 = tm * BM, c0 = tn * BN;
  const char* ga = (const char*)((const float*)p.A + batch * p.stride_a + (A_KF ? (int64_t)r0 * p.lda : (int64_t)r0));
  const char* gb = (const char*)((const float*)p.B + batch * p.stride_b + (B_KF ? (int64_t)c0 * p.ldb : (int64_t)c0));
  const int64_t a_step = A_KF ? (int64_t)128 : p.lda * (int64_t)(BK * 4);
  const int64_t b_step = B_KF ? (int64_t)128 : p.ldb * (int64_t)(BK * 4);
  // what lane `lane` of 1 KB load `id` (0 .. 7) of an operand's slab fetches: four values, the first of them at value
  // `k` of the slab; rows past the edge are clamped (extents along the contiguous index are multiples of 4)
  auto unit = [&](auto kf_c, int id, int64_t ld, int left, uint32_t& off, int& k) __attribute__((always_inline)) {
    if constexpr (decltype(kf_c)::value) {
      const int r = id * 8 + lane / 8, c = (lane % 8) ^ swz16(r);
      k = c * 4;
      off = (uint32_t)(((int64_t)min(r, left - 1) * ld + k) * 4);
    } else {
      const int line = lane >> 3, k8 = line ^ ((line >> 2) & 1);
      k = (id & 3) * 8 + k8;
      off = (uint32_t)(((int64_t)k * ld + min((id >> 2) * 32 + (lane & 7) * 4, left - 4)) * 4);
    }
  };
  typedef std::integral_constant<bool, A_KF> a_kf;
  typedef std::integral_constant<bool, B_KF> b_kf;
  uint32_t off[LOADS];
  int kf[LOADS];
#pragma unroll
  for (int q = 0; q < HALF; ++q) {
    unit(a_kf(), wave * HALF + q, p.lda, p.M - r0, off[q], kf[q]);
    unit(b_kf(), wave * HALF + q, p.ldb, p.N - c0, off[HALF + q], kf[HALF + q]);
  }
  const int T_full = p.K / BK, kvalid = p.K - T_full * BK;
  f32x4_t tail[LOADS];
  if (kvalid > 0) {                                     // requested first, multiplied last; zeros past K
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
      tail[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      const char* base = q < HALF ? ga + (int64_t)T_full * a_step : gb + (int64_t)T_full * b_step;
      if (kf[q] < kvalid) tail[q] = *(const f32x4_t*)(base + off[q]);
    }
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_uchar_t*)smem;
  auto uniform_ptr = [](const char* q) __attribute__((always_inline)) {
    const uint64_t gv = (uint64_t)q;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gv >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gv);
    return (const char*)(((uint64_t)hi << 32) | (uint64_t)lo);
  };
  auto issue = [&](int st) __attribute__((always_inline)) {
    const char* pa = uniform_ptr(ga);
    const char* pb = uniform_ptr(gb);
    const uint32_t la = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + st * STAGE + wave * (HALF * 1024)));
    asm volatile("s_nop 4" ::"s"(pa), "s"(pb), "s"(la));
#pragma unroll
    for (int q = 0; q < HALF; ++q)
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   ::"s"(la), "n"(q * 1024), "v"(off[q]), "s"(pa) : "memory", "m0", "scc");
#pragma unroll
    for (int q = 0; q < HALF; ++q)
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   ::"s"(la), "n"(A_BYTES + q * 1024), "v"(off[HALF + q]), "s"(pb) : "memory", "m0", "scc");
    ga += a_step;
    gb += b_step;
  };
  f32x16_t acc[MT][MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < MT; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.0f;
  // the lane's 16 values of a slab for the 32 rows from `row` on
  auto operand = [&](auto kf_c, const unsigned char* op, int row, float (&x)[16]) __attribute__((always_inline)) {
    if constexpr (decltype(kf_c)::value) {
      const int r = row + fr;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4_t t = *(const f32x4_t*)(op + r * 128 + (((2 * j + fh) ^ swz16(r)) * 16));
        x[4 * j] = t[0]; x[4 * j + 1] = t[1]; x[4 * j + 2] = t[2]; x[4 * j + 3] = t[3];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x[4 * j + e] = *(const float*)(op + ((row >> 5) * 4 + j) * 1024 + ((4 * fh + e) ^ fh) * 128 + fr * 4);
    }
  };
  auto multiply = [&](int st) __attribute__((always_inline)) {
    const unsigned char* s = smem + st * STAGE;
    float a[MT][16], w[MT][16];
#pragma unroll
    for (int m = 0; m < MT; ++m) operand(a_kf(), s, (wm * MT + m) * 32, a[m]);
#pragma unroll
    for (int n = 0; n < MT; ++n) operand(b_kf(), s + A_BYTES, (wn * MT + n) * 32, w[n]);
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < MT; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m][i], w[n][i], acc[m][n], 0, 0, 0);
  };
  const int ahead = NSTAGE - 1;
  for (int t = 0; t < ahead && t < T_full; ++t) issue(t);
  int st = 0;
  for (int t = 0; t < T_full; ++t) {
    if (t + ahead <= T_full) wait_vmcnt<(NSTAGE - 2) * LOADS>();   // slab t + 1, if there is one, may be on its way
    else wait_vmcnt<0>();
    wait_lgkmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (t + ahead < T_full) issue(st == 0 ? NSTAGE - 1 : st - 1);
    multiply(st);
    st = st + 1 == NSTAGE ? 0 : st + 1;
  }
  if (kvalid > 0) {
    wait_lgkmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < LOADS; ++q)
      *(f32x4_t*)(smem + (q < HALF ? 0 : A_BYTES) + (wave * HALF + q % HALF) * 1024 + lane * 16) = tail[q];
    __syncthreads();
    multiply(0);
  }
  // register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of the 32x32 tile
  const float* bias = p.has_bias ? p.bias + batch * p.stride_bias : nullptr;
  float* C = (float*)p.C + batch * p.stride_c;
#pragma unroll
  for (int n = 0; n < MT; ++n) {
    const int64_t j = c0 + (wn * MT + n) * 32 + fr;
    if (j >= p.N) continue;
    const float bj = bias ? bias[j] : 0.0f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t i = r0 + (wm * MT + m) * 32 + 8 * (r / 4) + 4 * fh + r % 4;
        if (i < p.M) C[i * c_si + j * c_sj] = apply_activation(p.act, acc[m][n][r] + bj, p.scale);
      }
  }
}

// ---- fp32 operands of any alignment and extent ----------------------------------------------------------------------
// The same tiles, LDS layout and products for operands that cannot be moved in aligned pieces of four values: the slabs travel
// global -> registers -> LDS in 16-byte loads that take four-byte alignment, two slabs on their way in registers and two in LDS, one
// barrier per slab.  Pieces that reach past K, and those of operands narrower than a tile, are put together element by
// element (moving them down from four values before the end by selects was slower: 1001^3, B row-major 52 us against 39).  Such problems ran on
// general_mfma_kernel, which loads single values in slabs of 16 columns of K: 1001^3, B row- / column-major 53.8 -> 39.0 / 54.3 -> 31.6 us,
// 3001^3 658 -> 506, 4001^3 1453 -> 1077 (119 TFLOP/s; 4000^3 takes 0.95 ms on f32_ring_kernel), 1518x587x2647 128 -> 66.
// ROWS: a lane holds values of one row of C (of one column otherwise): its neighbours' are next to each other in memory where C is
// column-major, or row-major with a few columns.
template <bool A_KF, bool B_KF, int MT, bool ROWS>
__global__ __launch_bounds__(256) void f32_any_kernel(MfmaArgs p, int64_t c_si, int64_t c_sj) {
  constexpr int BM = 64 * MT, BN = 64 * MT, BK = 32;
  constexpr int A_BYTES = BM * 128, STAGE = 2 * A_BYTES, HALF = 2 * MT, LOADS = 2 * HALF;
  struct __attribute__((packed, aligned(4))) Piece { f32x4_t v; };
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int fr = lane & 31, fh = lane >> 5;
  const int64_t batch = blockIdx.z;
  int tm, tn;
  tile_coords<false>(p, blockIdx.y * gridDim.x + blockIdx.x, p.tiles_m * p.tiles_n, tm, tn);
  // A K-strided operand's last tile ends with the last row, so that no piece reaches past it (the rows it shares with the tile before
  // are stored there); with fewer rows than a tile its pieces are put together element by element.
  const int row_first = tm * BM, col_first = tn * BN;
  const int r0 = A_KF ? row_first : min(row_first, max(p.M - BM, 0)), c0 = B_KF ? col_first : min(col_first, max(p.N - BN, 0));
  const char* ga = (const char*)((const float*)p.A + batch * p.stride_a + (A_KF ? (int64_t)r0 * p.lda : (int64_t)r0));
  const char* gb = (const char*)((const float*)p.B + batch * p.stride_b + (B_KF ? (int64_t)c0 * p.ldb : (int64_t)c0));
  const int64_t a_step = A_KF ? (int64_t)128 : p.lda * (int64_t)(BK * 4);
  const int64_t b_step = B_KF ? (int64_t)128 : p.ldb * (int64_t)(BK * 4);
  typedef std::integral_constant<bool, A_KF> a_kf;
  typedef std::integral_constant<bool, B_KF> b_kf;
  // the piece of four values that lane `lane` of load `id` fetches (f32_ring_kernel's): byte offset, first value of K, first row of the
  // piece (K strided; rows of K-contiguous operands are clamped)
  auto unit = [&](auto kf_c, int id, int64_t ld, int left, uint32_t& off, int& k, int& row) __attribute__((always_inline)) {
    if constexpr (decltype(kf_c)::value) {
      const int r = id * 8 + lane / 8, c = (lane % 8) ^ swz16(r);
      k = c * 4;
      row = 0;
      off = (uint32_t)(((int64_t)min(r, left - 1) * ld + k) * 4);
    } else {
      const int line = lane >> 3, k8 = line ^ ((line >> 2) & 1);
      k = (id & 3) * 8 + k8;
      row = (id >> 2) * 32 + (lane & 7) * 4;
      off = (uint32_t)(((int64_t)k * ld + row) * 4);
    }
  };
  uint32_t off[LOADS];
  {
    int k, row;
#pragma unroll
    for (int q = 0; q < HALF; ++q) {
      unit(a_kf(), wave * HALF + q, p.lda, p.M - r0, off[q], k, row);
      unit(b_kf(), wave * HALF + q, p.ldb, p.N - c0, off[HALF + q], k, row);
    }
  }
  // n valid values from `at` on, zeros behind them
  auto partial = [](const char* at, int n) __attribute__((always_inline)) {
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) v[e] = *(const float*)(at + e * 4);
    return v;
  };
  // one operand's pieces of a slab: whole inside the matrix; the last slab reaches past K
  auto load_op = [&](auto kf_c, f32x4_t* v, const uint32_t* at, const char* base, int k_left, int rows_left, int64_t ld) __attribute__((always_inline)) {
    constexpr bool kf = decltype(kf_c)::value;
    if (k_left >= BK && (kf || rows_left >= BM)) {
#pragma unroll
      for (int q = 0; q < HALF; ++q) v[q] = ((const Piece*)(base + at[q]))->v;
      return;
    }
#pragma unroll
    for (int q = 0; q < HALF; ++q) {
      uint32_t o; int k, row;
      unit(kf_c, wave * HALF + q, ld, rows_left, o, k, row);
      v[q] = partial(base + o, kf ? k_left - k : k < k_left ? rows_left - row : 0);
    }
  };
  f32x4_t v[2][LOADS];
  const int T = (p.K + BK - 1) / BK;
  auto load = [&](f32x4_t (&w)[LOADS], int t) __attribute__((always_inline)) {
    load_op(a_kf(), w, off, ga + (int64_t)t * a_step, p.K - t * BK, p.M - r0, p.lda);
    load_op(b_kf(), w + HALF, off + HALF, gb + (int64_t)t * b_step, p.K - t * BK, p.N - c0, p.ldb);
  };
  f32x16_t acc[MT][MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < MT; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.0f;
  auto operand = [&](auto kf_c, const unsigned char* op, int row, float (&x)[16]) __attribute__((always_inline)) {
    if constexpr (decltype(kf_c)::value) {
      const int r = row + fr;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4_t t = *(const f32x4_t*)(op + r * 128 + (((2 * j + fh) ^ swz16(r)) * 16));
        x[4 * j] = t[0]; x[4 * j + 1] = t[1]; x[4 * j + 2] = t[2]; x[4 * j + 3] = t[3];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x[4 * j + e] = *(const float*)(op + ((row >> 5) * 4 + j) * 1024 + ((4 * fh + e) ^ fh) * 128 + fr * 4);
    }
  };
  auto multiply = [&](int st) __attribute__((always_inline)) {
    const unsigned char* s = smem + st * STAGE;
    float a[MT][16], w[MT][16];
#pragma unroll
    for (int m = 0; m < MT; ++m) operand(a_kf(), s, (wm * MT + m) * 32, a[m]);
#pragma unroll
    for (int n = 0; n < MT; ++n) operand(b_kf(), s + A_BYTES, (wn * MT + n) * 32, w[n]);
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < MT; ++n)
          acc[m][n] = ROWS ? __builtin_amdgcn_mfma_f32_32x32x2f32(w[n][i], a[m][i], acc[m][n], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_32x32x2f32(a[m][i], w[n][i], acc[m][n], 0, 0, 0);
  };
  load(v[0], 0);
  if (T > 1) load(v[1], 1);
  for (int t0 = 0; t0 < T; t0 += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = t0 + u;
      if (t >= T) break;
      // (the stage was last read two slabs ago, a barrier in between)
#pragma unroll
      for (int q = 0; q < LOADS; ++q)
        *(f32x4_t*)(smem + u * STAGE + (q < HALF ? 0 : A_BYTES) + (wave * HALF + q % HALF) * 1024 + lane * 16) = v[u][q];
      wait_lgkmcnt<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (t + 2 < T) load(v[u], t + 2);
      multiply(u);
    }
  }
  // register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of the 32x32 tile (ROWS: the other way round)
  const float* bias = p.has_bias ? p.bias + batch * p.stride_bias : nullptr;
  float* C = (float*)p.C + batch * p.stride_c;
  if constexpr (ROWS) {
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int64_t i = r0 + (wm * MT + m) * 32 + fr;
      if (i >= p.M || i < row_first) continue;
#pragma unroll
      for (int n = 0; n < MT; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t j = c0 + (wn * MT + n) * 32 + 8 * (r / 4) + 4 * fh + r % 4;
          if (j < p.N && j >= col_first) C[i * c_si + j * c_sj] = apply_activation(p.act, acc[m][n][r] + (bias ? bias[j] : 0.0f), p.scale);
        }
    }
    return;
  }
#pragma unroll
  for (int n = 0; n < MT; ++n) {
    const int64_t j = c0 + (wn * MT + n) * 32 + fr;
    if (j >= p.N || j < col_first) continue;
    const float bj = bias ? bias[j] : 0.0f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t i = r0 + (wm * MT + m) * 32 + 8 * (r / 4) + 4 * fh + r % 4;
        if (i < p.M && i >= row_first) C[i * c_si + j * c_sj] = apply_activation(p.act, acc[m][n][r] + bj, p.scale);
      }
  }
}

}  // namespace mi355gemm
