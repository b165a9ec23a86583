// Matrix-core GEMM for few tiles and a long K (16-bit operands, both K-contiguous): every wave of a workgroup multiplies the whole
// tile over its own part of K.
//
// The ring kernel splits a tile over its waves, so that every value is read from LDS by several of them (64x64 tiles, 2x4 waves:
// 96 KB per 128 values of K, 32 KB of operands), and all waves meet at a barrier per slab.  Here wave w takes slabs w, w + WAVES, .. of
// 64 values into LDS of its own: each value is read once, and there is no barrier in the loop.  As soon as a slab's fragments are in
// registers the next one is requested over it.  At the end the waves' sums are added through LDS, in wave order.  What bounds it: the way
// from L2 (64 bytes per clock and CU) and its latency.  64x64 tiles have eight waves with one slab each (two waves per SIMD: one multiplies while
// the other waits), 32x32 tiles four waves with four.  Operands in the last-level cache / from HBM, against the ring kernel of the same tile:
// 512x2048x8192 30.2 -> 24.6 / 35.0 -> 30.3 us, 1024x1024x4096 17.0 -> 15.6 / 18.8 -> 17.1, 256x1024x4096 9.0 -> 8.0 / 10.4 -> 9.9.  Measured and not
// kept: 64x64 tiles with four waves and two slabs each (1024x1024x4096 16.4 / 18.5 us); tiles of 128x128 with four waves (2048x2048x4096 42 us,
// 30.6 on the four-slab kernel); fragments straight from global memory without LDS (1024x1024x4096 31.7).  Loads, swizzle and fragment order
// are those of ring_kernel.hpp; sums of more than one slab are added in another order.
#pragma once

#include "ring_kernel.hpp"

namespace mi355gemm {

template <int BM, int BN, int WAVES, int NSTAGE>
constexpr int kSplitLds = WAVES * (NSTAGE * (BM + BN) * 128 > BM * BN * 4 ? NSTAGE * (BM + BN) * 128 : BM * BN * 4);

template <typename T, int BM, int BN, int WAVES, int NSTAGE>
__global__ __launch_bounds__(64 * WAVES) void ksplit_ring_kernel(MfmaArgs p) {
  constexpr int MT = BM / 16, NT = BN / 16, E = (int)sizeof(T), EPC = 16 / E;
  constexpr int BK = 128 / E, AL = BM / 8, BL = BN / 8, LOADS = AL + BL, STAGE = (BM + BN) * 128;
  static_assert(E == 2 && NSTAGE <= 4 && (NSTAGE - 1) * LOADS <= 63 && kSplitLds<BM, BN, WAVES, NSTAGE> <= 160 * 1024, "");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kSplitLds<BM, BN, WAVES, NSTAGE>];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int batch, tm, tn;
  tile_and_batch<false>(p, batch, tm, tn);
  const int r0 = tm * BM, c0 = tn * BN;
  const char* ga = (const char*)((const T*)p.A + (int64_t)batch * p.stride_a + (int64_t)r0 * p.lda) + wave * 128;
  const char* gb = (const char*)((const T*)p.B + (int64_t)batch * p.stride_b + (int64_t)c0 * p.ldb) + wave * 128;

  // Load q of an operand fills 1 KB: 8 rows of 128 bytes (rows past the edge are clamped), 16-byte piece c of row r at slot c ^ swz16(r).
  auto piece = [&](int q) __attribute__((always_inline)) { return (lane % 8) ^ swz16(q * 8 + lane / 8); };
  uint32_t a_off[AL], b_off[BL];
#pragma unroll
  for (int q = 0; q < AL; ++q) a_off[q] = (uint32_t)((int64_t)min(q * 8 + lane / 8, p.M - 1 - r0) * p.lda * E) + (uint32_t)(piece(q) * 16);
#pragma unroll
  for (int q = 0; q < BL; ++q) b_off[q] = (uint32_t)((int64_t)min(q * 8 + lane / 8, p.N - 1 - c0) * p.ldb * E) + (uint32_t)(piece(q) * 16);
  unsigned char* const mine = smem + wave * (NSTAGE * STAGE);
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_uchar_t*)smem + wave * (NSTAGE * STAGE);
  auto uniform_ptr = [](const char* q) __attribute__((always_inline)) {
    const uint64_t gv = (uint64_t)q;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gv >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gv);
    return (const char*)(((uint64_t)hi << 32) | (uint64_t)lo);
  };
  // request the slab `ga` / `gb` point at into stage `st`, and move on to the wave's next one (M0: see ring_kernel.hpp)
  auto issue = [&](int st) __attribute__((always_inline)) {
    const char* pa = uniform_ptr(ga);
    const char* pb = uniform_ptr(gb);
    const uint32_t la = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + st * STAGE));
    asm volatile("s_nop 4" ::"s"(pa), "s"(pb), "s"(la));
#pragma unroll
    for (int q = 0; q < AL; ++q)
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   ::"s"(la), "n"(q * 1024), "v"(a_off[q]), "s"(pa) : "memory", "m0", "scc");
#pragma unroll
    for (int q = 0; q < BL; ++q)
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   ::"s"(la), "n"((AL + q) * 1024), "v"(b_off[q]), "s"(pb) : "memory", "m0", "scc");
    ga += WAVES * 128;
    gb += WAVES * 128;
  };

  f32x4acc_t acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = f32x4acc_t{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, fo = lane >> 4;
  auto frag = [&](const unsigned char* op, int row, int kk) __attribute__((always_inline)) {
    const int r = row + fr;
    return *(const u32x4_t*)(op + r * 128 + (((kk * 4 + fo) ^ swz16(r)) * 16));
  };
  u32x4_t af[MT][2], bf[NT][2];
  auto read = [&](int st, int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NT; ++n) bf[n][kk] = frag(mine + st * STAGE + BM * 128, n * 16, kk);
#pragma unroll
    for (int m = 0; m < MT; ++m) af[m][kk] = frag(mine + st * STAGE, m * 16, kk);
  };
  auto multiply = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[m][n] = Mfma16<T>::run(bf[n][kk], af[m][kk], acc[m][n]);
  };

  const int slabs = p.K / BK, kvalid = p.K - slabs * BK;
  const int count = slabs > wave ? (slabs - wave + WAVES - 1) / WAVES : 0;
  for (int i = 0; i < NSTAGE && i < count; ++i) issue(i);
  int st = 0;                                            // stage of slab i
  for (int i = 0; i < count; ++i) {
    // slab i has landed when at most the loads of the slabs requested after it are outstanding
    const int later = min(count - 1 - i, NSTAGE - 1);
    if (later == NSTAGE - 1) wait_vmcnt<(NSTAGE - 1) * LOADS>();
    else if (NSTAGE > 2 && later == NSTAGE - 2) wait_vmcnt<(NSTAGE > 2 ? NSTAGE - 2 : 0) * LOADS>();
    else if (NSTAGE > 3 && later == NSTAGE - 3) wait_vmcnt<(NSTAGE > 3 ? NSTAGE - 3 : 0) * LOADS>();
    else wait_vmcnt<0>();
    read(st, 0);
    read(st, 1);
    multiply(0);
    wait_lgkmcnt<0>();                                   // the fragments are in registers: the slab's LDS is free
    if (i + NSTAGE < count) issue(st);
    multiply(1);
    st = st + 1 == NSTAGE ? 0 : st + 1;
  }
  if (kvalid > 0 && wave == slabs % WAVES) {             // the K tail, the wave's next slab: pieces past K are zeros
    // (loaded here: where the built-in choice takes this kernel, only a leading dimension longer than K leaves a tail)
    const char* ta = ga - (int64_t)count * (WAVES * 128) + (int64_t)(slabs - wave) * 128;
    const char* tb = gb - (int64_t)count * (WAVES * 128) + (int64_t)(slabs - wave) * 128;
#pragma unroll
    for (int q = 0; q < AL; ++q) {
      u32x4_t v = {0u, 0u, 0u, 0u};
      if (piece(q) * EPC < kvalid) v = *(const u32x4_t*)(ta + a_off[q]);
      *(u32x4_t*)(mine + q * 1024 + lane * 16) = v;
    }
#pragma unroll
    for (int q = 0; q < BL; ++q) {
      u32x4_t v = {0u, 0u, 0u, 0u};
      if (piece(q) * EPC < kvalid) v = *(const u32x4_t*)(tb + b_off[q]);
      *(u32x4_t*)(mine + (AL + q) * 1024 + lane * 16) = v;
    }
    read(0, 0);
    read(0, 1);
    multiply(0);
    multiply(1);
  }

  // add the waves' sums (every wave is done with its slabs), each wave finishes its share of the 16x16 tiles
  __syncthreads();
  f32x4acc_t* sums = (f32x4acc_t*)smem;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) sums[(wave * MT * NT + m * NT + n) * 64 + lane] = acc[m][n];
  __syncthreads();
  const float* bias = p.has_bias ? p.bias + (int64_t)batch * p.stride_bias : nullptr;
  // (rows of C start at any element: the stores of four columns take element alignment)
  typedef f32x4_t __attribute__((aligned(4))) f32x4_any_t;
  typedef u32x2_t __attribute__((aligned(2))) u32x2_any_t;
  for (int t = wave; t < MT * NT; t += WAVES) {
    f32x4acc_t v = sums[t * 64 + lane];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) v += sums[(w * MT * NT + t) * 64 + lane];
    // lane l of a 16x16 tile holds row l % 16 and columns 4 (l / 16) .. +3 (operands go in swapped)
    const int i = r0 + t / NT * 16 + fr, j = c0 + t % NT * 16 + fo * 4;
    if (i >= p.M || j >= p.N) continue;
    const bool full = j + 3 < p.N;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = apply_activation(p.act, v[e] + (bias && j + e < p.N ? bias[j + e] : 0.0f), p.scale);
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
      T* c = (T*)p.C + o;
      if (full) {
        *(u32x2_any_t*)c = u32x2_t{pack2<T>(v[0], v[1]), pack2<T>(v[2], v[3])};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j + e < p.N) c[e] = from_float<T>(v[e]);
      }
    }
  }
}

}  // namespace mi355gemm
