// Matrix-core GEMM for problems that do not fill the chip with large tiles (16-bit or fp8 operands, fp32 accumulate):
// small tiles, NSTAGE slabs of K in a ring.
//
// What bounds these problems is latency: a slab of a large-tile kernel is requested while one earlier slab is
// multiplied, and with a tile or less per CU nothing else hides the 0.6 us a load takes (K = 4096: 64 slabs, 41 us,
// whatever M and N).  Here NSTAGE - 1 slabs are on their way while one is multiplied, a slab is KS * 128 bytes of K
// (one barrier for each), and the tiles are small enough that every CU has one.
// 64x6144x4096 bf16 41.0 -> 12.1 us, 32x6144x4096 40.5 -> 10.2, 64x4096x14336 133 -> 25, 1024^3 9.5 -> 6.7, 512^3
// 6.9 -> 3.6; fp8 64x6144x4096 15.4 -> 7.3.  What bounds it now: one turn of barrier, LDS reads and MFMAs per slab
// (0.23 to 0.45 us), and the L2 traffic of small tiles once every CU has two (15 - 23 TB/s).
// LDS layout, swizzle, fragment order and the direct-to-LDS loads are those of mfma16_kernel.hpp (slab = KS
// sub-slabs of 128 bytes of K); the fragment reads and their waits are left to the compiler, the loads' waits
// (vmcnt, in issue order) are placed by hand.
#pragma once

#include "mfma16_kernel.hpp"
#include "skinny_kernel.hpp"

namespace mi355gemm {

// One MFMA step on 16-byte (16-bit operands: 32 values of K) or 32-byte (fp8: 128 values of K) fragments per lane.
template <typename T> struct RingMfma {
  static constexpr int kParts = 1;
  static __device__ __forceinline__ f32x4acc_t run(const u32x4_t* a, const u32x4_t* b, f32x4acc_t c) {
    return Mfma16<T>::run(a[0], b[0], c);
  }
};
template <> struct RingMfma<f8e4m3_t> {
  static constexpr int kParts = 2;
  typedef int i32x8_t __attribute__((ext_vector_type(8)));
  static __device__ __forceinline__ i32x8_t join(const u32x4_t* v) {
    return __builtin_bit_cast(i32x8_t, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
  }
  // both formats E4M3, no block scaling; which 32 of the step's 128 values of K a lane holds is free as long as
  // both operands agree, so the two halves are those of two consecutive 16-bit steps
  static __device__ __forceinline__ f32x4acc_t run(const u32x4_t* a, const u32x4_t* b, f32x4acc_t c) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(join(a), join(b), c, 0, 0, 0, 0, 0, 0);
  }
};

template <typename T, int BM, int BN, int WM, int WN, int KS, int NSTAGE>
struct RingTile {
  static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
  static constexpr int WTM = BM / WM, WTN = BN / WN, MT = WTM / 16, NT = WTN / 16;
  static constexpr int BK = KS * 128 / (int)sizeof(T);          // values of K per slab
  static constexpr int A_LOADS = KS * BM / 8 / kWaves, B_LOADS = KS * BN / 8 / kWaves, LOADS = A_LOADS + B_LOADS;
  static constexpr int A_BYTES = KS * BM * 128, B_BYTES = KS * BN * 128, STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES;
  static_assert(A_LOADS * 8 * kWaves == KS * BM && B_LOADS * 8 * kWaves == KS * BN, "loads divide over the waves");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0 && LDS_BYTES <= 160 * 1024, "");
  static_assert((NSTAGE - 1) * LOADS <= 63, "outstanding loads fit the counter");
};

// A_KF, B_KF: K is the contiguous index of A / B (16-bit operands may have it strided: see mfma16_gemm_kernel)
// DIRECT = false: rows, extents and pointers of any alignment (two bytes), C in either layout.  The same slabs travel
// global -> registers -> LDS, the next one or two requested while one is multiplied: 16-byte loads at two-byte alignment
// inside the matrix, element by element in the last slab's pieces that reach past K.  Such problems ran on
// the fp32 matrix-core instruction, element by element: 4001^3 bf16 2413 -> 204 us, B row-major 2510 -> 235 us,
// 1000x1000x1001 83 -> 15 us.
template <typename T, typename TO, int BM, int BN, int WM, int WN, int KS, int NSTAGE, bool A_KF, bool B_KF, bool DIRECT = true>
__global__ __launch_bounds__(64 * WM * WN) void ring_gemm_kernel(MfmaArgs p) {
  typedef RingTile<T, BM, BN, WM, WN, KS, NSTAGE> Cfg;
  constexpr int MT = Cfg::MT, NT = Cfg::NT, LOADS = Cfg::LOADS, E = (int)sizeof(T);
  constexpr int P = RingMfma<T>::kParts;               // 64-byte steps of K per MFMA
  constexpr int EPC = 16 / E;                           // values per 16-byte piece
  static_assert((A_KF && B_KF) || E == 2, "strided operands: 16-bit only");
  static_assert((A_KF || BM % 64 == 0) && (B_KF || BN % 64 == 0), "K-strided operands: blocks of 64 rows");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[Cfg::LDS_BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  int batch, tm, tn;
  tile_and_batch<kEitherOrder<BM, BN, NSTAGE, false>>(p, batch, tm, tn);
  const int r0 = tm * BM, c0 = tn * BN;
  // K-strided operands of any alignment are addressed from a row that has eight behind it (where there are eight)
  const int ra = DIRECT || A_KF ? r0 : min(r0, max(p.M - 8, 0)), rb = DIRECT || B_KF ? c0 : min(c0, max(p.N - 8, 0));
  const char* ga = (const char*)((const T*)p.A + (int64_t)batch * p.stride_a + (A_KF ? (int64_t)ra * p.lda : (int64_t)ra));
  const char* gb = (const char*)((const T*)p.B + (int64_t)batch * p.stride_b + (B_KF ? (int64_t)rb * p.ldb : (int64_t)rb));
  const int64_t a_step = A_KF ? (int64_t)(KS * 128) : p.lda * (int64_t)(Cfg::BK * E);
  const int64_t b_step = B_KF ? (int64_t)(KS * 128) : p.ldb * (int64_t)(Cfg::BK * E);

  // Load q of this wave fills 1 KB of a sub-slab: 8 rows of 128 bytes (K contiguous) or 8 values of K x 64 rows;
  // rows past the edge are clamped.  kfirst: the first value of K (within the slab) the lane's piece holds; row: the
  // first row (within the tile) of a piece of 8 rows.
  auto a_unit = [&](int q, int ln, uint32_t& off, int& kfirst, int& row) __attribute__((always_inline)) {
    const int id = wave * Cfg::A_LOADS + q, ks = id / (BM / 8), blk = id % (BM / 8);
    if constexpr (A_KF) {
      const int r = blk * 8 + ln / 8, c = (ln % 8) ^ swz16(r);
      kfirst = (ks * 8 + c) * EPC;
      row = 0;
      off = (uint32_t)((int64_t)min(r, p.M - 1 - r0) * p.lda * E) + (uint32_t)(ks * 128 + c * 16);
    } else {
      const int kg = blk & 7, j8 = ln >> 3, key = ((j8 >> 1) & 1) | ((kg & 1) << 1);
      kfirst = ks * 64 + kg * 8 + j8;
      row = (blk >> 3) * 64 + ((ln & 7) ^ (key * 2)) * 8;
      off = (uint32_t)(((int64_t)kfirst * p.lda + (DIRECT ? min(row, p.M - 8 - r0) : min(r0 + row, max(p.M - 8, 0)) - ra)) * 2);
    }
  };
  auto b_unit = [&](int q, int ln, uint32_t& off, int& kfirst, int& row) __attribute__((always_inline)) {
    const int id = wave * Cfg::B_LOADS + q, ks = id / (BN / 8), blk = id % (BN / 8);
    if constexpr (B_KF) {
      const int r = blk * 8 + ln / 8, c = (ln % 8) ^ swz16(r);
      kfirst = (ks * 8 + c) * EPC;
      row = 0;
      off = (uint32_t)((int64_t)min(r, p.N - 1 - c0) * p.ldb * E) + (uint32_t)(ks * 128 + c * 16);
    } else {
      const int kg = blk & 7, j8 = ln >> 3, key = ((j8 >> 1) & 1) | ((kg & 1) << 1);
      kfirst = ks * 64 + kg * 8 + j8;
      row = (blk >> 3) * 64 + ((ln & 7) ^ (key * 2)) * 8;
      off = (uint32_t)(((int64_t)kfirst * p.ldb + (DIRECT ? min(row, p.N - 8 - c0) : min(c0 + row, max(p.N - 8, 0)) - rb)) * 2);
    }
  };
  uint32_t a_off[Cfg::A_LOADS], b_off[Cfg::B_LOADS];
  {
    int unused, unused2;
#pragma unroll
    for (int q = 0; q < Cfg::A_LOADS; ++q) a_unit(q, lane, a_off[q], unused, unused2);
#pragma unroll
    for (int q = 0; q < Cfg::B_LOADS; ++q) b_unit(q, lane, b_off[q], unused, unused2);
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_uchar_t*)smem;
  auto uniform_ptr = [](const char* q) __attribute__((always_inline)) {
    const uint64_t gv = (uint64_t)q;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gv >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gv);
    return (const char*)(((uint64_t)hi << 32) | (uint64_t)lo);
  };
  // request slab `ga`/`gb` point at into stage `st`, and move on (M0 takes the LDS address; a scalar register
  // written by the vector unit must be five wait states old before a load reads it: the s_nop covers the read-back)
  auto issue = [&](int st) __attribute__((always_inline)) {
    const char* pa = uniform_ptr(ga);
    const char* pb = uniform_ptr(gb);
    const uint32_t la = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + st * Cfg::STAGE_BYTES + wave * (Cfg::A_LOADS * 1024)));
    const uint32_t lb = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + st * Cfg::STAGE_BYTES + Cfg::A_BYTES + wave * (Cfg::B_LOADS * 1024)));
    asm volatile("s_nop 4" ::"s"(pa), "s"(pb), "s"(la), "s"(lb));
#pragma unroll
    for (int q = 0; q < Cfg::A_LOADS; ++q)
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   ::"s"(la), "n"(q * 1024), "v"(a_off[q]), "s"(pa) : "memory", "m0", "scc");
#pragma unroll
    for (int q = 0; q < Cfg::B_LOADS; ++q)
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   ::"s"(lb), "n"(q * 1024), "v"(b_off[q]), "s"(pb) : "memory", "m0", "scc");
    ga += a_step;
    gb += b_step;
  };

  f32x4acc_t acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = f32x4acc_t{0.f, 0.f, 0.f, 0.f};

  // Fragment of 16 rows, 64-byte step kk of the slab: lane l holds row l % 16, 16-byte piece l / 16 of the step
  // (K contiguous), or the same values gathered by two transposing reads.
  const int fr = lane & 15, fo = lane >> 4;
  auto frag = [&](auto kf_c, const unsigned char* op, int rows, int row, int kk) __attribute__((always_inline)) {
    const unsigned char* sub = op + (kk >> 1) * (rows * 128);
    if constexpr (decltype(kf_c)::value) {
      const int r = row + fr;
      return *(const u32x4_t*)(sub + r * 128 + ((((kk & 1) * 4 + fo) ^ swz16(r)) * 16));
    } else {
      typedef short s16x4_t __attribute__((ext_vector_type(4)));
      typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
      const int j = fr >> 2, key = ((j >> 1) & 1) | ((fo & 1) << 1);
      const unsigned char* at = sub + (row >> 6) * 8192 + ((kk & 1) * 4 + fo) * 1024 + j * 128 + ((((row >> 4) & 3) ^ key) * 32) + (fr & 3) * 8;
      const u32x2_t lo = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)at));
      const u32x2_t hi = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(at + 512)));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
    }
  };
  auto multiply = [&](int st) __attribute__((always_inline)) {
    const unsigned char* sa = smem + st * Cfg::STAGE_BYTES;
    const unsigned char* sb = sa + Cfg::A_BYTES;
#pragma unroll
    for (int kk = 0; kk < 2 * KS; kk += P) {
      u32x4_t af[MT][P], bf[NT][P];
#pragma unroll
      for (int h = 0; h < P; ++h) {
#pragma unroll
        for (int m = 0; m < MT; ++m) af[m][h] = frag(std::integral_constant<bool, A_KF>(), sa, BM, wm * Cfg::WTM + m * 16, kk + h);
#pragma unroll
        for (int n = 0; n < NT; ++n) bf[n][h] = frag(std::integral_constant<bool, B_KF>(), sb, BN, wn * Cfg::WTN + n * 16, kk + h);
      }
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[m][n] = RingMfma<T>::run(bf[n], af[m], acc[m][n]);
    }
  };

  if constexpr (!DIRECT) {
    struct __attribute__((packed, aligned(2))) Piece { u32x4_t v; };
    // Slabs on their way: two for 64x64 tiles of K-contiguous operands (84x678x16089 182 -> 139 us, 150x4843x5511 68 -> 52, 1000x1000x1001 17.0 ->
    // 14.6), one for 128x128 tiles and K-strided operands, whose registers allow fewer workgroups with two (4001^3 200 -> 212, B row-major 231
    // -> 298).
    constexpr int AHEAD = A_KF && B_KF && BM == 64 ? 2 : 1;
    u32x4_t av[AHEAD][Cfg::A_LOADS], bv[AHEAD][Cfg::B_LOADS];
    // n valid values from `at` on, zeros behind them
    auto partial = [](const char* at, int n) __attribute__((always_inline)) {
      uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e < n) w[e >> 1] |= (uint32_t)*(const uint16_t*)(at + e * 2) << (16 * (e & 1));
      return u32x4_t{w[0], w[1], w[2], w[3]};
    };
    // One operand's pieces of slab t.  K contiguous: only the last slab reaches past K.  K strided: a piece that
    // reaches past the last row is read from eight rows before the end and moved down (what ends up in rows past the
    // edge does not matter, their results are dropped); values of K past the end are zeros.
    auto load_op = [&](auto kf_c, auto loads_c, u32x4_t* v, const uint32_t* off_in, const char* base, int left, int rows, int first,
                       auto unit) __attribute__((always_inline)) {
      constexpr bool kf = decltype(kf_c)::value;
      constexpr int loads = decltype(loads_c)::value;
      constexpr int tile = loads * 8 * Cfg::kWaves / KS;
      if (left >= Cfg::BK && (kf || first + tile <= rows)) {
#pragma unroll
        for (int q = 0; q < loads; ++q) v[q] = ((const Piece*)(base + off_in[q]))->v;
        return;
      }
#pragma unroll
      for (int q = 0; q < loads; ++q) {
        uint32_t off; int k, row;
        unit(q, lane, off, k, row);
        if constexpr (kf) {
          v[q] = partial(base + off, left - k);
        } else if (rows < 8) {
          v[q] = partial(base + off, k < left ? rows - first - row : 0);
        } else {
          unsigned __int128 w = 0;
          if (k < left) w = __builtin_bit_cast(unsigned __int128, ((const Piece*)(base + off))->v);
          v[q] = __builtin_bit_cast(u32x4_t, w >> (16 * min(7, max(0, first + row - (rows - 8)))));
        }
      }
    };
    auto load = [&](u32x4_t* va, u32x4_t* vb, int t) __attribute__((always_inline)) {
      const int left = p.K - t * Cfg::BK;
      load_op(std::integral_constant<bool, A_KF>(), std::integral_constant<int, Cfg::A_LOADS>(), va, a_off, ga + (int64_t)t * a_step, left, p.M, r0, a_unit);
      load_op(std::integral_constant<bool, B_KF>(), std::integral_constant<int, Cfg::B_LOADS>(), vb, b_off, gb + (int64_t)t * b_step, left, p.N, c0, b_unit);
    };
    const int T_all = (p.K + Cfg::BK - 1) / Cfg::BK;
    auto stash = [&](int st, const u32x4_t* va, const u32x4_t* vb) __attribute__((always_inline)) {
      unsigned char* to = smem + st * Cfg::STAGE_BYTES;              // (last read two slabs ago, a barrier in between)
#pragma unroll
      for (int q = 0; q < Cfg::A_LOADS; ++q) *(u32x4_t*)(to + (wave * Cfg::A_LOADS + q) * 1024 + lane * 16) = va[q];
#pragma unroll
      for (int q = 0; q < Cfg::B_LOADS; ++q) *(u32x4_t*)(to + Cfg::A_BYTES + (wave * Cfg::B_LOADS + q) * 1024 + lane * 16) = vb[q];
    };
    load(av[0], bv[0], 0);
    if constexpr (AHEAD == 1) {
      for (int t = 0; t < T_all; ++t) {
        stash(t & 1, av[0], bv[0]);
        __syncthreads();
        if (t + 1 < T_all) load(av[0], bv[0], t + 1);
        multiply(t & 1);
      }
    } else {
      if (T_all > 1) load(av[1], bv[1], 1);
      for (int t0 = 0; t0 < T_all; t0 += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int t = t0 + u;
          if (t >= T_all) break;
          stash(u, av[u], bv[u]);
          wait_lgkmcnt<0>();
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          if (t + 2 < T_all) load(av[u], bv[u], t + 2);
          multiply(u);
        }
      }
    }
  } else {
  const int T_full = p.K / Cfg::BK;
  const int ahead = NSTAGE - 1;
  // K tail: requested before everything else and kept in registers, so that its latency (3 us at the end of a call
  // that takes 10) is hidden behind the slabs.  Pieces past K are zeros.
  const int kvalid = p.K - T_full * Cfg::BK;
  u32x4_t ta[Cfg::A_LOADS], tb[Cfg::B_LOADS];
  if (kvalid > 0) {
    const char* pa = ga + (int64_t)T_full * a_step;
    const char* pb = gb + (int64_t)T_full * b_step;
#pragma unroll
    for (int q = 0; q < Cfg::A_LOADS; ++q) {
      uint32_t off; int k, row;
      a_unit(q, lane, off, k, row);
      ta[q] = u32x4_t{0u, 0u, 0u, 0u};
      if (k < kvalid) ta[q] = *(const u32x4_t*)(pa + off);
    }
#pragma unroll
    for (int q = 0; q < Cfg::B_LOADS; ++q) {
      uint32_t off; int k, row;
      b_unit(q, lane, off, k, row);
      tb[q] = u32x4_t{0u, 0u, 0u, 0u};
      if (k < kvalid) tb[q] = *(const u32x4_t*)(pb + off);
    }
  }
  for (int t = 0; t < ahead && t < T_full; ++t) issue(t);
  int st = 0;                                            // stage of slab t
  for (int t = 0; t < T_full; ++t) {
    // slab t has landed when at most the loads of the slabs requested after it are outstanding
    const int later = min(T_full - 1 - t, ahead - 1);
    if (later == ahead - 1) wait_vmcnt<(NSTAGE - 2) * LOADS>();
    else if (NSTAGE > 3 && later == ahead - 2) wait_vmcnt<(NSTAGE > 3 ? NSTAGE - 3 : 0) * LOADS>();
    else if (NSTAGE > 4 && later == ahead - 3) wait_vmcnt<(NSTAGE > 4 ? NSTAGE - 4 : 0) * LOADS>();
    else wait_vmcnt<0>();
    wait_lgkmcnt<0>();                                   // own reads of slab t - 1 are done
    __builtin_amdgcn_s_barrier();                        // so are everyone's: its stage is free
    asm volatile("" ::: "memory");
    if (t + ahead < T_full) issue(st == 0 ? NSTAGE - 1 : st - 1);
    multiply(st);
    st = st + 1 == NSTAGE ? 0 : st + 1;
  }
  if (kvalid > 0) {                                      // the K tail, in stage 0
    wait_lgkmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < Cfg::A_LOADS; ++q) *(u32x4_t*)(smem + (wave * Cfg::A_LOADS + q) * 1024 + lane * 16) = ta[q];
#pragma unroll
    for (int q = 0; q < Cfg::B_LOADS; ++q) *(u32x4_t*)(smem + Cfg::A_BYTES + (wave * Cfg::B_LOADS + q) * 1024 + lane * 16) = tb[q];
    __syncthreads();
    multiply(0);
  }
  }

  // Lane l of a 16x16 accumulator tile holds row l % 16 and columns 4 (l / 16) .. +3 (operands go in swapped).
  const float* bias = p.has_bias ? p.bias + (int64_t)batch * p.stride_bias : nullptr;
  // (rows of C start at any element: the stores of four columns take element alignment)
  typedef f32x4_t __attribute__((aligned(4))) f32x4_any_t;
  typedef u32x2_t __attribute__((aligned(2))) u32x2_any_t;
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int j = c0 + wn * Cfg::WTN + n * 16 + fo * 4;
    if (j >= p.N) continue;
    float bv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) bv[e] = bias && j + e < p.N ? bias[j + e] : 0.0f;
    const bool full = j + 3 < p.N;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int i = r0 + wm * Cfg::WTM + m * 16 + fr;
      if (i >= p.M) continue;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = apply_activation(p.act, acc[m][n][e] + bv[e], p.scale);
      if (!DIRECT && p.c_col) {                        // a lane's columns are ldc apart
        const int64_t o = (int64_t)batch * p.stride_c + i + j * p.ldc;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (j + e >= p.N) break;
          if (p.c_f32) ((float*)p.C)[o + e * p.ldc] = v[e];
          else ((TO*)p.C)[o + e * p.ldc] = from_float<TO>(v[e]);
        }
        continue;
      }
      const int64_t o = (int64_t)batch * p.stride_c + (int64_t)i * p.ldc + j;
      if (p.c_f32) {
        float* c = (float*)p.C + o;
        if (full) {
          *(f32x4_any_t*)c = f32x4_t{v[0], v[1], v[2], v[3]};
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j + e < p.N) c[e] = v[e];
        }
      } else {
        TO* c = (TO*)p.C + o;
        if (full) {
          *(u32x2_any_t*)c = u32x2_t{pack2<TO>(v[0], v[1]), pack2<TO>(v[2], v[3])};
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j + e < p.N) c[e] = from_float<TO>(v[e]);
        }
      }
    }
  }
}

}  // namespace mi355gemm
