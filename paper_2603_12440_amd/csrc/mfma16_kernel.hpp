// Matrix-core GEMM for gfx950 on the 16x16x32 MFMA shape: 16-bit operands (bf16 / fp16), fp32 accumulate; and on the 16x16x128
// shape: 8-bit floating point (OCP E4M3).
//
//   C = act(A . B + bias),  A row-major (K contiguous), B column-major (K contiguous: the
//   "weight" matrix stored N x K), C row-major; also A column-major and / or B row-major.
//
// Same data path as mfma_kernel.hpp (direct-to-LDS slabs of 64 columns of K, two stages,
// XOR-swizzled 16-byte chunks, 16-byte fragment reads, accumulators in AccVGPRs, hand-placed
// waits), but the products are issued as v_mfma_f32_16x16x32: measured on an MI355X, whose
// matrix pipes are power-limited, that shape delivers about a tenth more FLOP/s than
// v_mfma_f32_32x32x16 at the same power (it reads and writes a quarter of the accumulator
// registers per instruction and sums 32 products before touching them).  What else differs:
//   * a k-step is 32 columns of K and is multiplied in G sub-steps of MT/G row fragments
//     times all NT column fragments, so that the fragment registers are double-buffered per
//     sub-step (A) and per k-step (B) instead of per whole k-step of both;
//   * the global -> LDS loads of a slab are spread over the sub-steps that follow the
//     hand-over instead of being issued in one burst;
//   * with two waves per SIMD, each wave lowers its priority as it advances from one
//     hand-over to the next, so that the wave that is behind gets the matrix pipe and the
//     two alternate sub-step by sub-step instead of one running ahead to the barrier.
// fp8: the same slabs, loads and reads in bytes; a slab row of 128 values is one k-step, multiplied in G = 4 sub-steps.  A lane's 32
// values are the two pieces that two k-steps of 16-bit values would read.  The column fragments are not double-buffered: the last
// sub-step runs column by column, and each fragment of the next slab is requested behind the last MFMA that takes the registers it
// goes to, so a wave needs no more fragment registers (64) than with 16-bit operands.  Bound by power: an MFMA-only loop runs at 4.3
// PFLOP/s (32x32x64: 4.0, with the same error), 8192^3 with operands from HBM takes 358 us = 3.07 PFLOP/s.  The kernel that this
// one replaced (32x32x64, one tile per workgroup, no prefetch): 8192^3 401 us, 4096x12288x4096 156, 4096^3 52.6 against 49.2, 128x128
// tiles 486 against 467.  Measured here: loads over one or three sub-steps 383 / 368 us, no prefetch 371 (operands in the
// last-level cache: 346 without it, 350 with it).
// Paper taxonomy (Sec. 3.2): d_mem = 3, d_algo = 1 (fused post-op), d_sync = 1.
#pragma once

#include <type_traits>

#include "mfma_kernel.hpp"

namespace mi355gemm {

// kStep: values of K one MFMA takes; kParts: 16-byte LDS reads per fragment and lane where K is contiguous.  (fp8: 32 values of K
// per lane in two pieces 64 values apart; which of a step's values a lane holds is free as long as A and B agree.)
template <typename T> struct Frag16;
template <> struct Frag16<bf16_t> {
  static constexpr int kStep = 32, kParts = 1;
  static __device__ __forceinline__ void mfma(const u32x4_t& x, const u32x4_t& y, f32x4_t& c) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
  }
};
template <> struct Frag16<f16_t> {
  static constexpr int kStep = 32, kParts = 1;
  static __device__ __forceinline__ void mfma(const u32x4_t& x, const u32x4_t& y, f32x4_t& c) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
  }
};
typedef uint32_t u32x8_t __attribute__((ext_vector_type(8)));
template <> struct Frag16<f8e4m3_t> {
  static constexpr int kStep = 128, kParts = 2;
  // (both operand formats default to fp8 E4M3, no block scaling)
  static __device__ __forceinline__ void mfma(const u32x8_t& x, const u32x8_t& y, f32x4_t& c) {
    asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
  }
};

// Chunk c (16 bytes) of slab row r is stored at chunk slot c ^ swz16(r).  A fragment read
// touches 16 consecutive rows at one logical chunk per quarter wave; rows are 128 bytes
// apart (32 banks), so row parity picks the half of the banks and (r >> 1) & 7 the 16-byte
// slot within it: the 16 rows cover all 64 banks once.  The key uses row bits 1..3 only, so
// fragments 16 rows apart differ by a constant offset.
__device__ __forceinline__ int swz16(int r) { return (r >> 1) & 7; }

// ---- the instruction order of one sub-step, generated at compile time ---------------------
// A sub-step multiplies MA row fragments with NT column fragments.  While it runs, the reads
// for the next sub-step are requested, one behind each of its first MFMAs: MA row fragments
// and, when the next sub-step begins a new k-step, the NT column fragments too (WITH_B).
// Its own MFMAs run in the order in which their operands were requested one sub-step earlier.
// RA, RB: LDS reads per row / column fragment (one 16-byte read, or two 8-byte transposing ones).
// COLS: the MFMAs run column by column (the last sub-step of a slab of one k-step, whose column fragments are overwritten one by one).
template <int MA, int NT, bool WITH_B, int RA, int RB, bool COLS = false>
struct SubOrder {
  static constexpr int kReads = MA * RA + (WITH_B ? NT * RB : 0), kMfma = MA * NT;
  struct Tables {
    int r_isb[kReads], r_idx[kReads], r_part[kReads];
    int mm[kMfma], nn[kMfma];
    int need[kMfma];        // request position of the later of MFMA i's operands (-1: resident)
  };
  static constexpr Tables make() {
    Tables t{};
    int pos_a[MA] = {}, pos_b[NT] = {};
    for (int n = 0; n < NT; ++n) pos_b[n] = -1;
    int c = 0;
    auto ask_a = [&](int i) { for (int q = 0; q < RA; ++q) { t.r_isb[c] = 0; t.r_idx[c] = i; t.r_part[c] = q; pos_a[i] = c++; } };
    auto ask_b = [&](int i) { for (int q = 0; q < RB; ++q) { t.r_isb[c] = 1; t.r_idx[c] = i; t.r_part[c] = q; pos_b[i] = c++; } };
    if (WITH_B) {
      // a0 b0 b1 a1 b2 a2 ...: the first MFMAs can start after two fragments
      for (int i = 0; i < (MA > NT ? MA : NT); ++i) {
        if (i == 0) {
          ask_a(0);
          ask_b(0);
        } else {
          if (i < NT) ask_b(i);
          if (i < MA) ask_a(i);
        }
      }
    } else {
      for (int i = 0; i < MA; ++i) ask_a(i);
    }
    bool used[kMfma] = {};
    for (int i = 0; i < kMfma; ++i) {
      int best = -1, best_key = 0;
      for (int q = 0; q < kMfma; ++q) {
        if (used[q]) continue;
        const int m = q / NT, n = q % NT;
        const int p = pos_a[m] > pos_b[n] ? pos_a[m] : pos_b[n];
        const int key = (p + 1) * kMfma + q + (COLS ? n * (kReads + 2) * kMfma : 0);
        if (best < 0 || key < best_key) { best = q; best_key = key; }
      }
      used[best] = true;
      t.mm[i] = best / NT;
      t.nn[i] = best % NT;
      t.need[i] = (best_key / kMfma) % (kReads + 2) - 1;
    }
    return t;
  }
  static constexpr Tables t = make();
};
// Behind which MFMA of a sub-step of type Ord each of its requests for the next one (OrdN) goes out: spread over the first MFMAs; a
// column fragment (KEEP) not before the last MFMA that takes what its registers hold.  at[]: ascending; before[i]: requests ahead of
// MFMA i.
template <typename Ord, typename OrdN, bool KEEP>
struct ReadSlots {
  struct Tables { int at[OrdN::kReads], before[Ord::kMfma + 1]; };
  static constexpr Tables make() {
    Tables t{};
    constexpr int per_mfma = (OrdN::kReads + Ord::kMfma - 1) / Ord::kMfma;
    int from = 0;
    for (int r = 0; r < OrdN::kReads; ++r) {
      int at = KEEP ? 0 : r / per_mfma;
      if (KEEP && OrdN::t.r_isb[r])
        for (int i = 0; i < Ord::kMfma; ++i)
          if (Ord::t.nn[i] == OrdN::t.r_idx[r] && i > at) at = i;
      from = at > from ? at : from;
      t.at[r] = from;
    }
    for (int i = 0; i <= Ord::kMfma; ++i)
      for (int r = 0; r < OrdN::kReads; ++r) t.before[i] += t.at[r] < i ? 1 : 0;
    return t;
  }
  static constexpr Tables t = make();
};

template <typename T, int BM, int BN, int WM, int WN, int G, int STAGES = 2, bool A_KF = true>
struct Mfma16Tile {
  static constexpr int ES = (int)sizeof(T), BK = 128 / ES, NSTAGE = STAGES;
  static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
  static constexpr int WTM = BM / WM, WTN = BN / WN;     // per-wave block
  static constexpr int MT = WTM / 16, NT = WTN / 16;     // 16x16 MFMA tiles per wave
  static constexpr int MA = (MT + G - 1) / G;            // row fragments per sub-step, at most
  static constexpr int group_rows(int g) { return (MT + G - 1 - g) / G; }      // of sub-step g of a k-step (7 = 4 + 3)
  static constexpr int group_first(int g) { return g == 0 ? 0 : group_first(g - 1) + group_rows(g - 1); }
  static constexpr int KK = BK / Frag16<T>::kStep;       // k-steps per slab: two, fp8 one
  static constexpr int NSUB = KK * G;                    // sub-steps per slab
  static constexpr int ROWB = BK * ES;                   // bytes per slab row
  static constexpr int CPR = ROWB / 16, RPI = 64 / CPR;  // chunks per row, rows per wave-wide load
  // A wave-wide load fills 8 rows of A's slab; where those do not divide over the waves, the waves take them in turn and the last
  // ones issue one load less.  (A K-strided A is stored in blocks of 64 rows: BM is a multiple.)
  static constexpr int A_UNITS = BM / RPI, A_LOADS = (A_UNITS + kWaves - 1) / kWaves, B_LOADS = BN / RPI / kWaves;
  static constexpr bool UNEVEN = A_UNITS % kWaves != 0;
  static constexpr int A_ID_WAVE = UNEVEN ? 1 : A_LOADS, A_ID_Q = UNEVEN ? kWaves : 1;    // load q of a wave is unit wave * A_ID_WAVE + q * A_ID_Q
  static constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES;
  // the epilogue's staging area of a persistent workgroup: one 16-row band of every wave's block in fp32
  static constexpr int EPI_BYTES = kWaves * 16 * WTN * 4;
  // Prefetch into L2 (see the kernel): two slabs in LDS and one workgroup per CU.  What the prefetches write to LDS lands
  // in 256 bytes behind the slabs that nothing reads (a persistent workgroup: in the staging area, idle during the K loop).
  static constexpr bool PREFETCH = NSTAGE == 2 && kWaves == 8;
  static constexpr int DUMP_BYTES = PREFETCH ? 256 : 0;
  static_assert(ES == 2 || A_KF, "8-bit operands are K-contiguous");
  static_assert(BM % (8 * RPI) == 0 || BM % 32 == 0, "whole wave-wide loads");
  static_assert(A_KF || BM % 64 == 0, "a K-strided A is stored in blocks of 64 rows");
  static_assert(BN % (RPI * kWaves) == 0, "slab rows of B must divide over waves");
  static_assert(!UNEVEN || (NSTAGE == 2 && A_LOADS == B_LOADS), "the load that some waves leave out is the last of a slab's second half");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0 && MT >= G, "wave block in whole sub-steps");
  static_assert(NSUB % 2 == 0, "the row-fragment double buffer alternates per sub-step");
  static_assert(KK == 1 || group_rows(G - 1) * NT >= MA + NT, "a sub-step issues one or two fragment reads behind each MFMA");
  static_assert(LDS_BYTES + (STAGES == 2 ? EPI_BYTES : 0) <= 160 * 1024, "LDS budget");
};

// The fragment registers of one operand: one 16-byte LDS read (K contiguous in memory; fp8: two) or two 8-byte
// transposing reads, each four of the lane's eight values of K (K strided).
template <typename T, bool KF> struct FragReg {
  u32x4_t h[1];
  __device__ __forceinline__ u32x4_t get() const { return h[0]; }
};
template <> struct FragReg<f8e4m3_t, true> {
  u32x4_t h[2];
  __device__ __forceinline__ u32x8_t get() const { return __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7); }
};
template <typename T> struct FragReg<T, false> {
  u32x2_t h[2];
  __device__ __forceinline__ u32x4_t get() const { return __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3); }
};
// Four 16-bit values per lane out of a 4 x 16 block per 16 lanes, transposed on the way: lane i of the 16
// passes the address of values 4 (i % 4) .. +3 of row i / 4 and receives value i of the rows 0 .. 3.
template <typename F>
__device__ __forceinline__ void lds_read_tr16(F& dst, uint32_t addr, int offset) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(offset) : "memory");
}

// T: operand type; TO: the 16-bit output type (outputs may also be fp32: MfmaArgs::c_f32).
// PERSIST: a workgroup walks over several tiles (tile ids blockIdx.x, blockIdx.x + gridDim.x,
// ...) as one software pipeline: the slabs of the next tile are requested while the last slabs
// of the current one are multiplied, and land while its epilogue runs, which stages C through an
// LDS region of its own.  Needs K to be a whole number of slabs, at least two.
// A_KF, B_KF: K is the contiguous index of A / of B in memory (A row-major, B column-major).  An operand
// whose rows (A) or columns (B) are contiguous instead keeps that order in LDS: its slab is stored as
// 1 KB blocks of 8 values of K x 64 rows (block = 8 * (row / 64) + k / 8, 128 bytes per value of K), so that
// the direct-to-LDS loads still read whole 128-byte lines, and the fragments are read with
// ds_read_b64_tr_b16, which transposes 4 x 16 blocks on the way to the registers.  The 32-byte piece
// (16 rows) t of value k sits at piece t ^ key(k), key = bit 1 of k and (as bit 1) bit 3 of k: a read touches
// 4 values of K per 16 lanes, whose 128-byte rows alternate between the halves of the banks, and the key
// spreads the remaining factor of 4 over the pieces of a half.
// Bound like the K-contiguous variant (power and matrix pipes: the same bytes, loads and MFMAs per slab, twice
// the LDS read instructions at half the width): 8192^3 bf16 takes 721 us with B row-major, 726 us with A
// column-major as well, 709 - 726 us K-contiguous on the same box.  These layouts used to run on the fp32
// matrix-core instruction: 6144 x 4096 x 3001 with both operands strided 2475 us, here 118 us.
// S: slabs in LDS.  Two for the large problems; a lone workgroup on a CU has nothing else to hide a load's latency
// behind and takes four (one tile per workgroup only).
template <typename T, typename TO, int BM, int BN, int WM, int WN, int G, bool PERSIST, bool A_KF = true, bool B_KF = true, int S = 2>
__global__ __launch_bounds__(64 * WM * WN) void mfma16_gemm_kernel(MfmaArgs p) {
  typedef Mfma16Tile<T, BM, BN, WM, WN, G, S, A_KF> Cfg;
  static_assert(S == 2 || !PERSIST, "a persistent workgroup streams through two stages");
  constexpr int MT = Cfg::MT, NT = Cfg::NT, MA = Cfg::MA, CPR = Cfg::CPR, RPI = Cfg::RPI;
  constexpr int ROWB = Cfg::ROWB, BK = Cfg::BK, KK = Cfg::KK, NSUB = Cfg::NSUB;
  constexpr bool kEither = kEitherOrder<BM, BN, S, PERSIST>;
  constexpr bool kTwoPerSimd = Cfg::kWaves > 4;          // two waves share a SIMD: alternate by priority
  constexpr int ES = Cfg::ES, EPC = 16 / ES;             // bytes per value, values per 16-byte piece
  constexpr int RA = A_KF ? Frag16<T>::kParts : 2, RB = B_KF ? Frag16<T>::kParts : 2;    // LDS reads per fragment
  static_assert((B_KF || (BN % 64 == 0 && Cfg::WTN % 64 == 0)) && ((A_KF && B_KF) || BK == 64),
                "K-strided operands are stored in blocks of 64 rows x 8 values of K");
  // bytes from one slab of an operand to the next
  const int64_t a_step = A_KF ? (int64_t)ROWB : p.lda * (int64_t)(BK * 2);
  const int64_t b_step = B_KF ? (int64_t)ROWB : p.ldb * (int64_t)(BK * 2);
  // K-strided operand: what lane `ln` of load `id` of a slab fetches (8 rows from `row` on of value `k`)
  auto strided_unit = [](int id, int ln, int& k, int& row) __attribute__((always_inline)) {
    const int kg = id & 7, j8 = ln >> 3, key = ((j8 >> 1) & 1) | ((kg & 1) << 1);
    k = kg * 8 + j8;
    row = (id >> 3) * 64 + ((ln & 7) ^ (key * 2)) * 8;
  };

  __shared__ __attribute__((aligned(1024))) unsigned char smem[Cfg::LDS_BYTES + (PERSIST ? Cfg::EPI_BYTES : Cfg::DUMP_BYTES)];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // which 1 KB of A's slab this wave's load q fills, and whether there is such a piece
  auto a_unit = [&](int q) __attribute__((always_inline)) { return wave * Cfg::A_ID_WAVE + q * Cfg::A_ID_Q; };
  auto has_unit = [&](int q) __attribute__((always_inline)) { return !Cfg::UNEVEN || q < Cfg::A_LOADS - 1 || a_unit(q) < Cfg::A_UNITS; };
  // One tile per workgroup: the batch is the grid's second index.  A persistent workgroup walks over
  // the tiles of every problem of the batch (tile id = problem * n_tiles + tile within the problem);
  // `batch` is then the problem of the tile being written out.
  int batch = PERSIST ? 0 : (int)blockIdx.y;
  const int n_tiles = p.tiles_m * p.tiles_n;
  const int total_tiles = PERSIST ? n_tiles * p.batches : n_tiles;
  // A batch on persistent workgroups (xcd_remap == 2; grid and tile count multiples of 8): the 8 XCDs
  // (round-robin dispatch: XCD = tile id mod 8) each take a contiguous run of the problems, so that the
  // tiles of one problem, which share its panels, meet in one L2 instead of fetching them 8 times.
  auto logical_tile = [&](const MfmaArgs& p, int vid) __attribute__((always_inline)) {
    return p.xcd_remap == 2 ? (vid & 7) * (total_tiles >> 3) + (vid >> 3) : vid;
  };
  // What finding a tile's panels needs of the arguments.  A persistent workgroup reads them from the argument block again for
  // every tile but its first (the kernel's only argument sits at the start of the kernarg segment), so that they do not occupy
  // scalar registers during the K loops.
  typedef __attribute__((address_space(4))) const volatile MfmaArgs kernarg_t;
  auto tile_args = [&]() __attribute__((always_inline)) {
    MfmaArgs q = p;
    if constexpr (PERSIST) {
      kernarg_t* pv = (kernarg_t*)__builtin_amdgcn_kernarg_segment_ptr();
      q.A = pv->A; q.B = pv->B; q.M = pv->M; q.N = pv->N; q.lda = pv->lda; q.ldb = pv->ldb;
      q.stride_a = pv->stride_a; q.stride_b = pv->stride_b; q.tiles_m = pv->tiles_m; q.tiles_n = pv->tiles_n;
      q.order.div_group = pv->order.div_group; q.order.div_rows = pv->order.div_rows; q.order.div_h = pv->order.div_h;
      q.xcd_remap = pv->xcd_remap; q.touch = pv->touch;
    }
    return q;
  };

  // ---- global -> LDS addressing (as in mfma_kernel.hpp, with this kernel's swizzle) -------
  // Load q of this wave fills LDS bytes [slab + (wave*LOADS + q)*1024, +1024): lane l writes
  // 16 bytes at +16*l, i.e. slab row (wave*LOADS+q)*RPI + l/CPR, slot l%CPR, which must
  // receive logical chunk slot ^ swz16(row).  Rows past the matrix edge are clamped to the
  // last valid row (their results are never stored).
  // The tile the loads work on (it runs ahead of the tile being multiplied):
  const char* ld_a;                              // first byte of the next slab to request, A and B
  const char* ld_b;
  uint32_t a_off[Cfg::A_LOADS], b_off[Cfg::B_LOADS];
  // Prefetch: a slab's loads have less than one slab's time to land in LDS, which is not enough for lines that come from HBM
  // (4096x3072x6144: 148 us with operands from HBM, 117 from the last-level cache).  So once per slab each wave touches
  // lines of the next slab but one, ahead of the loads that will want them; waves of the lower half touch A's, the others
  // B's.  The touch is a 4-byte load per lane into an LDS area nobody reads, so that no register is written later; it is the
  // youngest load at the hand-over, which leaves it in flight.  A panel is shared by the tiles that one XCD works on at a
  // time (A's by 4, B's by 8, or as many as there are: tile_order.hpp), so each workgroup touches its share of the 128-byte
  // lines only: 512 lines per workgroup and slab, all of them, cost 2.5 % where the operands are cached, this share 1 to 2 %.
  // (A quarter of the lines whatever the number of tiles left most of B untouched where there are few tile rows: 192x57344x4096
  // 126 us, 119 this way; 512x28672x4096 108 / 97, 300x57344x2048 102 / 86, 64 x (512x512x256) 19.6 / 17.2; short batches with
  // cached operands lose up to 3 %: 60 x (256x1024x512) 20.2 / 20.9.)
  // Operands from HBM: 4096x3072x6144 148 -> 127 us, 4096x4096x6144 158 -> 144, 8192^3 748 -> 737; touching two or three
  // slabs ahead is no better (8192^3: 718 / 723 / 726).
  constexpr bool PF = Cfg::PREFETCH;
  uint32_t pf_off = 0;                           // this lane's line within its operand's slab
  const bool pf_a = wave < Cfg::kWaves / 2;
  int ld_tm, ld_tn, ld_batch;                    // which tile that is, of which problem
  auto locate = [&](const MfmaArgs& p, int vid) __attribute__((always_inline)) {
    const int n_tiles = p.tiles_m * p.tiles_n;
    if constexpr (PERSIST) {
      const int lid = logical_tile(p, vid);
      ld_batch = lid / n_tiles;
      tile_coords<kEither>(p, lid - ld_batch * n_tiles, n_tiles, ld_tm, ld_tn);
    } else if constexpr (S == 2) {
      ld_batch = batch;
      tile_coords<kEither>(p, vid, n_tiles, ld_tm, ld_tn);
    } else {
      tile_and_batch<kEither>(p, ld_batch, ld_tm, ld_tn);
    }
  };
  // Leaves ld_a / ld_b at slab `kt` of that tile.  (`ln`: the lane id; a persistent workgroup recomputes the offsets from a fresh
  // copy of it after each epilogue, so that they need not stay in registers across it.)
  auto load_tile = [&](const MfmaArgs& p, int ln, int kt) __attribute__((always_inline)) {
    const int tm = ld_tm, tn = ld_tn, lb = ld_batch;
    const int r0 = tm * BM, c0 = tn * BN;
    if constexpr (PF) {
      // Lines of a slab: one per row where K is contiguous, else one per value of K and 64 rows.
      const int wave_lines = 2 * (pf_a ? BM : BN) / Cfg::kWaves;
      const int line = (wave % (Cfg::kWaves / 2)) * wave_lines +
                       touched_line(ln, pf_a ? tn : tm, pf_a ? p.touch & 15 : p.touch >> 4, wave_lines);
      const int64_t ld = pf_a ? p.lda : p.ldb;
      const int left = pf_a ? p.M - r0 : p.N - c0;
      auto row_line = [&]() __attribute__((always_inline)) { return (uint32_t)((int64_t)min(line, left - 1) * ld * ES); };
      auto k_line = [&](int per_k) __attribute__((always_inline)) {
        return (uint32_t)(((int64_t)(line / per_k) * ld + min(line % per_k * 64, left - 8)) * 2);
      };
      if constexpr (A_KF && B_KF) pf_off = row_line();
      else if (pf_a) pf_off = A_KF ? row_line() : k_line(BM / 64);
      else pf_off = B_KF ? row_line() : k_line(BN / 64);
    }
    ld_a = (const char*)((const T*)p.A + (int64_t)lb * p.stride_a + (A_KF ? (int64_t)r0 * p.lda : (int64_t)r0)) + (int64_t)kt * a_step;
    ld_b = (const char*)((const T*)p.B + (int64_t)lb * p.stride_b + (B_KF ? (int64_t)c0 * p.ldb : (int64_t)c0)) + (int64_t)kt * b_step;
#pragma unroll
    for (int q = 0; q < Cfg::A_LOADS; ++q) {
      if constexpr (!A_KF) {                      // (M is a multiple of 8 here: a unit of 8 rows is never split)
        int k, row;
        strided_unit(a_unit(q), ln, k, row);
        a_off[q] = (uint32_t)(((int64_t)k * p.lda + min(row, p.M - 8 - r0)) * 2);
        continue;
      }
      const int r = a_unit(q) * RPI + ln / CPR;
      const int c = (ln % CPR) ^ swz16(r);
      const int rr = min(r, p.M - 1 - r0);
      a_off[q] = (uint32_t)(((int64_t)rr * p.lda + c * EPC) * ES);
    }
#pragma unroll
    for (int q = 0; q < Cfg::B_LOADS; ++q) {
      if constexpr (!B_KF) {
        int k, row;
        strided_unit(wave * Cfg::B_LOADS + q, ln, k, row);
        b_off[q] = (uint32_t)(((int64_t)k * p.ldb + min(row, p.N - 8 - c0)) * 2);
        continue;
      }
      const int r = (wave * Cfg::B_LOADS + q) * RPI + ln / CPR;
      const int c = (ln % CPR) ^ swz16(r);
      const int rr = min(r, p.N - 1 - c0);
      b_off[q] = (uint32_t)(((int64_t)rr * p.ldb + c * EPC) * ES);
    }
  };
  locate(p, blockIdx.x);
  load_tile(p, lane, 0);
  const char* const Ab = ld_a;                   // (the first tile's panels: the one-tile path indexes them by slab)
  const char* const Bb = ld_b;

  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_uchar_t*)smem;
  constexpr int kLoads = Cfg::A_LOADS + Cfg::B_LOADS;
  // Where the loads of one slab go and come from: the slab's first byte in A and in B and the
  // LDS addresses of this wave's share of the stage's A and B parts.  All four are wave-uniform
  // and are read back through the scalar unit once per slab, far from the loads that use them.
  struct SlabIo { const char* ga; const char* gb; uint32_t la, lb; };
  auto uniform_ptr = [](const char* q) __attribute__((always_inline)) {
    const uint64_t gv = (uint64_t)q;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gv >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gv);
    return (const char*)(((uint64_t)hi << 32) | (uint64_t)lo);
  };
  auto slab_io_at = [&](const char* ga, const char* gb, int st) __attribute__((always_inline)) {
    SlabIo io;
    io.ga = uniform_ptr(ga);
    io.gb = uniform_ptr(gb);
    io.la = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + st * Cfg::STAGE_BYTES + wave * (Cfg::A_ID_WAVE * 1024)));
    io.lb = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(lds_base + st * Cfg::STAGE_BYTES + Cfg::A_BYTES + wave * (Cfg::B_LOADS * 1024)));
    return io;
  };
  auto slab_io = [&](int kt, int st) __attribute__((always_inline)) {
    return slab_io_at(Ab + (int64_t)kt * a_step, Bb + (int64_t)kt * b_step, st);
  };
  // One direct-to-LDS load (scalar base + 32-bit lane offset; M0 = LDS destination of the wave,
  // lane l lands at M0 + 16*l): q < A_LOADS fills the A slab, the rest the B slab.  M0 is written
  // by a scalar add; one wait state must pass before the load reads it.  The address pair must
  // not have been written by a vector instruction within five cycles of the load (the hardware
  // does not check): slab_io produces it long before, and the build scans the generated code for it.
  // (UNEVEN: B's loads go first, so that the load some waves leave out is the last of the slab.)
  auto issue_one_load = [&](int i, const SlabIo& io) __attribute__((always_inline)) {
    const int q = Cfg::UNEVEN ? (i + Cfg::A_LOADS) % kLoads : i;
    if (q < Cfg::A_LOADS) {
      if (!has_unit(q)) return;
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   :: "s"(io.la), "n"(q * Cfg::A_ID_Q * 1024), "v"(a_off[q < Cfg::A_LOADS ? q : 0]), "s"(io.ga) : "memory", "m0", "scc");
    } else {
      asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                   :: "s"(io.lb), "n"((q - Cfg::A_LOADS) * 1024), "v"(b_off[q >= Cfg::A_LOADS ? q - Cfg::A_LOADS : 0]), "s"(io.gb) : "memory", "m0", "scc");
    }
  };

  // this wave's prefetch of the slab at ga / gb
  auto prefetch = [&](const char* ga, const char* gb) __attribute__((always_inline)) {
    const char* g = uniform_ptr(pf_a ? ga : gb);
    // (a persistent workgroup: the wave's own staging buffer, as other waves may still be in the last tile's epilogue)
    const uint32_t dump = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(lds_base + Cfg::LDS_BYTES + (PERSIST ? wave * (Cfg::EPI_BYTES / Cfg::kWaves) : 0)));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" :: "s"(dump), "v"(pf_off), "s"(g) : "memory", "m0");
  };

  // K tail: chunks past K must read as zero, which a direct-to-LDS load cannot do, so that one
  // slab goes through registers.  (K is a multiple of 8 where an operand's K is contiguous: chunks are never split.)
  // The four-wave tiles have the registers to request it before the first slab (PRE), which hides its latency.
  constexpr bool PRE = !PERSIST && Cfg::kWaves == 4 && BM * BN <= 128 * 128;
  u32x4_t tail_v[kLoads];
  auto load_tail_q = [&](int kt, int q) __attribute__((always_inline)) {
    const int kvalid = p.K - kt * BK;
    u32x4_t v = {0u, 0u, 0u, 0u};
    if (q < Cfg::A_LOADS) {
      const int r = a_unit(q) * RPI + lane / CPR;
      int k = ((lane % CPR) ^ swz16(r)) * EPC, row = 0;            // the piece's first value of K
      if constexpr (!A_KF) strided_unit(a_unit(q), lane, k, row);
      if (k < kvalid) v = *(const u32x4_t*)(Ab + (int64_t)kt * a_step + a_off[q < Cfg::A_LOADS ? q : 0]);
    } else {
      const int qb = q >= Cfg::A_LOADS ? q - Cfg::A_LOADS : 0;
      const int r = (wave * Cfg::B_LOADS + qb) * RPI + lane / CPR;
      int k = ((lane % CPR) ^ swz16(r)) * EPC, row = 0;
      if constexpr (!B_KF) strided_unit(wave * Cfg::B_LOADS + qb, lane, k, row);
      if (k < kvalid) v = *(const u32x4_t*)(Bb + (int64_t)kt * b_step + b_off[qb]);
    }
    return v;
  };
  auto store_tail_q = [&](int q, const u32x4_t& v) __attribute__((always_inline)) {       // into stage 0
    if (q < Cfg::A_LOADS && !has_unit(q)) return;
    unsigned char* to = q < Cfg::A_LOADS ? smem + a_unit(q) * 1024
                                         : smem + Cfg::A_BYTES + wave * (Cfg::B_LOADS * 1024) + (q - Cfg::A_LOADS) * 1024;
    *(u32x4_t*)(to + lane * 16) = v;
  };

  // ---- LDS -> fragment addressing ---------------------------------------------------------
  // MFMA 16x16x32 operand: lane l holds 8 consecutive k of row (l % 16), k-octet l / 16 of the
  // step's four.  (fp8: pieces l / 16 and 4 + l / 16 of the row, what two steps of 16-bit values would read.)  Fragment m of the wave is 16*m rows further on: a constant offset.  The
  // address registers point into the stage being read and move to the other stage at each
  // hand-over (one vector add each), so a fragment read needs no address arithmetic.
  // (K-strided operand: one register for each of the four 32-byte pieces of a 64-row block, see A_KF.)
  constexpr int NA = A_KF ? 2 : 4, NB = B_KF ? 2 : 4;
  uint32_t a_rd[NA], b_rd[NB];
  int rd_delta;                                  // to the other stage (alternates in sign)
  // point the address registers into stage `st` (`ln`: the lane id, see load_tile)
  auto set_read_stage = [&](int st, int ln) __attribute__((always_inline)) {
    const int fr = ln & 15, fo = ln >> 4;
    const int a_row = wm * Cfg::WTM + fr;
    const int b_row = wn * Cfg::WTN + fr;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int c = kk * 4 + fo;
      if constexpr (A_KF) a_rd[kk] = lds_base + st * Cfg::STAGE_BYTES + a_row * ROWB + ((c ^ swz16(a_row)) * 16);
      if constexpr (B_KF) b_rd[kk] = lds_base + st * Cfg::STAGE_BYTES + Cfg::A_BYTES + b_row * ROWB + ((c ^ swz16(b_row)) * 16);
    }
    if constexpr (!A_KF || !B_KF) {
      const int j = fr >> 2, key = ((j >> 1) & 1) | ((fo & 1) << 1);
      const int at = lds_base + st * Cfg::STAGE_BYTES + fo * 1024 + j * 128 + (fr & 3) * 8;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        // (fragment m of the wave is the 32-byte piece f % 4 of block f / 4, f = wm * MT + m; x = m % 4)
        if constexpr (!A_KF) a_rd[x] = at + ((wm * MT + x) >> 2) * 8192 + ((((wm * MT + x) & 3) ^ key) * 32);
        if constexpr (!B_KF) b_rd[x] = at + Cfg::A_BYTES + (wn * Cfg::WTN / 64) * 8192 + ((x ^ key) * 32);
      }
    }
    rd_delta = st == S - 1 ? -(S - 1) * Cfg::STAGE_BYTES : Cfg::STAGE_BYTES;
  };
  set_read_stage(0, lane);
  auto flip_read_stage = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < NA; ++x) a_rd[x] += rd_delta;
#pragma unroll
    for (int x = 0; x < NB; ++x) b_rd[x] += rd_delta;
    if constexpr (S == 2) rd_delta = -rd_delta;
  };

  f32x4_t acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[m][n][r] = 0.0f;
  // The MFMAs are assembly statements the compiler's hazard recogniser cannot see: all zeros are written here, well before the
  // first product (left to itself the compiler put a register's zero right in front of the MFMA that reads it, which then
  // took the old value).
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) asm volatile("" : "+a"(acc[m][n]));
  asm volatile("s_nop 7" ::: "memory");

  // Fragment registers: row fragments double-buffered per sub-step, column fragments per k-step.
  // (One k-step per slab, KK == 1: one set of column fragments, each overwritten behind the last MFMA of the slab that takes it.)
  FragReg<T, A_KF> af[2][MA];
  FragReg<T, B_KF> bf[KK][NT];

  // Sub-step u of a slab: k-step u / G, row group u % G.
  // the i-th read of the requests made for sub-step `u` (from the stage the address registers point into)
  auto read_one = [&](auto u_c, int i) __attribute__((always_inline)) {
    constexpr int u = decltype(u_c)::value;
    constexpr int kk = u / G, g = u % G;
    typedef SubOrder<Cfg::group_rows(g), NT, g == 0, RA, RB> Ord;
    const int idx = Ord::t.r_idx[i], part = Ord::t.r_part[i];
    if (Ord::t.r_isb[i]) {
      if constexpr (B_KF) lds_read_b128(bf[kk][idx].h[part], b_rd[KK == 1 ? part : kk], idx * (16 * ROWB));
      else lds_read_tr16(bf[kk][idx].h[part], b_rd[idx & 3], (idx >> 2) * 8192 + kk * 4096 + part * 512);
    } else {
      const int m = Cfg::group_first(g) + idx;
      if constexpr (A_KF) lds_read_b128(af[u & 1][idx].h[part], a_rd[KK == 1 ? part : kk], m * (16 * ROWB));
      else lds_read_tr16(af[u & 1][idx].h[part], a_rd[m & 3], (m >> 2) * 8192 + kk * 4096 + part * 512);
    }
  };
  auto read_all = [&](auto u_c) __attribute__((always_inline)) {
    constexpr int u = decltype(u_c)::value;
    typedef SubOrder<Cfg::group_rows(u % G), NT, (u % G) == 0, RA, RB> Ord;
#pragma unroll
    for (int i = 0; i < Ord::kReads; ++i) read_one(u_c, i);
  };

  // One sub-step `u`: its MFMAs in the order their operands were requested, preceded by the
  // wait they need (LDS reads return in order; a wait is only issued when an MFMA needs a later
  // request than every MFMA before it); with `reads`, the requests for the next sub-step go out
  // one behind each of the first MFMAs; loads q0 .. q1-1 of the slab `io` are spaced evenly
  // over the MFMAs.
  auto sub_step = [&](auto u_c, bool reads, int q0, int q1, const SlabIo& io, bool do_loads = true) __attribute__((always_inline)) {
    constexpr int u = decltype(u_c)::value;
    constexpr int kk = u / G, g = u % G;
    constexpr int un = (u + 1) % NSUB;                    // the sub-step the reads are for
    constexpr bool keep = KK == 1 && un == 0;             // the requests overwrite column fragments in use
    typedef SubOrder<Cfg::group_rows(g), NT, g == 0, RA, RB, keep> Ord;   // how this sub-step's operands were requested
    typedef SubOrder<Cfg::group_rows(un % G), NT, (un % G) == 0, RA, RB> OrdN; // this sub-step's own requests
    typedef ReadSlots<Ord, OrdN, keep> Slots;
    const int nq = q1 - q0;
    int waited = -1;
#pragma unroll
    for (int i = 0; i < Ord::kMfma; ++i) {
      const int m = Ord::t.mm[i], n = Ord::t.nn[i];
      if (Ord::t.need[i] > waited) {
        // since the needed request: the rest of that sub-step's requests and those of ours so far
        const int after = (Ord::kReads - 1 - Ord::t.need[i]) + (reads ? Slots::t.before[i] : 0);
        wait_lgkmcnt_dyn(after);                 // (the counter holds 15 at most: larger values wait for 15)
        waited = Ord::t.need[i];
      }
      Frag16<T>::mfma(bf[kk][n].get(), af[u & 1][m].get(), acc[Cfg::group_first(g) + m][n]);
#pragma unroll
      for (int r = 0; r < OrdN::kReads; ++r)
        if (reads && Slots::t.at[r] == i) read_one(std::integral_constant<int, un>(), r);
#pragma unroll
      for (int j = 0; j < nq; ++j)
        if ((int)((j + 0.5f) * Ord::kMfma / nq) == i) {
          if (do_loads) issue_one_load(q0 + j, io);      // (a wave-uniform branch around one statement)
        }
    }
  };
  auto set_prio = [&](int pr) __attribute__((always_inline)) {
    if (!kTwoPerSimd) return;
    switch (pr) {
      case 0: __builtin_amdgcn_s_setprio(0); break;
      case 1: __builtin_amdgcn_s_setprio(1); break;
      case 2: __builtin_amdgcn_s_setprio(2); break;
      default: __builtin_amdgcn_s_setprio(3); break;
    }
  };

  // ---- epilogue of the tile at (row0, col0) ---------------------------------------------------
  auto epilogue = [&](int row0, int col0) __attribute__((always_inline)) {
    // What the epilogue needs of the arguments.  A persistent workgroup reads them from the argument
    // block again for every tile (the kernel's only argument sits at the start of the kernarg segment),
    // so that they do not occupy scalar registers during the K loops.
    MfmaArgs pe = p;
    if constexpr (PERSIST) {
      kernarg_t* pv = (kernarg_t*)__builtin_amdgcn_kernarg_segment_ptr();
      pe.C = pv->C; pe.bias = pv->bias; pe.M = pv->M; pe.N = pv->N; pe.ldc = pv->ldc; pe.stride_c = pv->stride_c;
      pe.stride_bias = pv->stride_bias; pe.has_bias = pv->has_bias; pe.act = pv->act; pe.c_f32 = pv->c_f32;
      pe.c_cached = pv->c_cached; pe.scale = pv->scale;
    }
    // The MFMAs were issued through inline assembly: the compiler inserts none of the wait states
    // a vector-ALU read of a just-written MFMA result needs.  Wait once, and route every
    // accumulator through an (empty) volatile statement placed after the wait.
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) asm volatile("" : "+a"(acc[m][n]));

    // ---- epilogue ---------------------------------------------------------------------------
    // Lane l of a 16x16 accumulator tile holds row (l % 16) and, in its four registers, columns
    // 4*(l / 16) .. +3 (the operands go in swapped, column fragment first).  For whole-line
    // stores each wave passes one 16-row band of its block at a time through its own piece of
    // the (now idle) LDS: 8- or 16-byte writes in accumulator order, 16-byte reads in row order.
    const float* bias = pe.has_bias ? pe.bias + (int64_t)batch * pe.stride_bias : nullptr;
    const int act = pe.act;
    auto fresh_lane = []() __attribute__((always_inline)) {
      unsigned z = 0;
      asm volatile("" : "+v"(z));
      return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, z));
    };
    const int elane = fresh_lane();
    const int er = elane & 15, eq = elane >> 4;

    // bias of the 4 columns j .. j+3 (zero past N; j is a multiple of 4); 16-byte loads only when the
    // bias vector of this batch starts at a 16-byte aligned address (the same for every lane)
    const bool bias_vec = (((uintptr_t)bias) & 15) == 0;
    auto bias4 = [&](int j, float (&bv)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[e] = 0.0f;
      if (!bias) return;
      if (j + 3 < pe.N && bias_vec) {
        const f32x4_t b4 = *(const f32x4_t*)(bias + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[e] = b4[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j + e < pe.N) bv[e] = bias[j + e];
      }
    };

    // Rows of C start at any element: the 16-byte stores take element alignment.  (Element by element where rows
    // were not whole 16-byte pieces: 2432x2431x4096 60 us, 51 this way; 3000x9001x256 62 and 37.)
    typedef u32x4_t __attribute__((aligned(2))) u32x4_any_t;
    typedef f32x4_t __attribute__((aligned(4))) f32x4_any_t;
    constexpr int OROWB = Cfg::WTN * 2;           // bytes per 16-bit row of the wave's block (128 or 256)
    constexpr int CH = OROWB / 16;
    constexpr int kShare = Cfg::LDS_BYTES / Cfg::kWaves;
    static_assert(OROWB == 128 || OROWB == 192 || OROWB == 256, "staging rows of 128, 192 or 256 bytes");
    static_assert(2 * 16 * OROWB <= (PERSIST ? Cfg::EPI_BYTES / Cfg::kWaves : kShare), "two 16-bit bands per wave");
    // staging: this wave's share of the idle slab stages, or of the separate area of a persistent workgroup
    unsigned char* wt = PERSIST ? smem + Cfg::LDS_BYTES + wave * (Cfg::EPI_BYTES / Cfg::kWaves) : smem + wave * kShare;
    // chunk-slot key of staging row r: 128-byte rows alternate between the two halves of the banks, 192-byte rows
    // start at each quarter in turn, 256-byte rows all start at bank 0; within groups of 4 chunks where a row is no power of two
    auto osw = [](int r) __attribute__((always_inline)) { return OROWB == 128 ? ((r >> 1) & 7) : OROWB == 192 ? (r >> 2) & 3 : (r & 15); };

    // 16-bit through LDS, pipelined over the 16-row bands of the wave block with two staging
    // buffers: while the rows of band m-1 come back from LDS, the values of band m+1 are computed;
    // a band's stores are on their way to memory while the next one is drained.
    constexpr int kBand16 = 16 * OROWB;             // bytes of one staged band
    constexpr int kIt16 = 16 * CH / 64;             // wave-wide 16-byte accesses per band
    auto drain16_all = [&](auto actf) __attribute__((always_inline)) {
      TO* Cb = (TO*)pe.C + (int64_t)batch * pe.stride_c;
      const int slane = fresh_lane();
      u32x2_t w[NT];
      u32x4_t val[kIt16];
      float bvs[NT][4];                           // the bias of this lane's columns, the same for every band
#pragma unroll
      for (int n = 0; n < NT; ++n) bias4(col0 + wn * Cfg::WTN + n * 16 + eq * 4, bvs[n]);
      auto values = [&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = actf(acc[m][n][e] + bvs[n][e]);
          w[n] = u32x2_t{pack2<TO>(v[0], v[1]), pack2<TO>(v[2], v[3])};
        }
      };
      auto write = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const int q = n * 2 + (eq >> 1);
          *(u32x2_t*)(wt + buf * kBand16 + er * OROWB + ((q ^ osw(er)) * 16) + (eq & 1) * 8) = w[n];
        }
      };
      auto read = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kIt16; ++it) {
          const int e = it * 64 + slane;
          const int r = e / CH, q = e % CH;
          val[it] = *(const u32x4_t*)(wt + buf * kBand16 + r * OROWB + ((q ^ osw(r)) * 16));
        }
      };
      // A tile that lies wholly inside C (the common case) stores without per-element tests, from a
      // wave-uniform base with 32-bit lane offsets: the epilogue is bound by instruction issue (two
      // waves per SIMD drain 128 accumulators each), so every address and mask instruction counts.
      const bool inside = row0 + BM <= pe.M && col0 + BN <= pe.N && (int64_t)BM * pe.ldc * 2 < ((int64_t)1 << 31);
      char* const wave_c = (char*)(Cb + (int64_t)(row0 + wm * Cfg::WTM) * pe.ldc + col0 + wn * Cfg::WTN);
      const uint32_t band_step = (uint32_t)(16 * pe.ldc * 2);
      uint32_t lane_off[kIt16];
#pragma unroll
      for (int it = 0; it < kIt16; ++it) {
        const int e = it * 64 + slane;
        lane_off[it] = (uint32_t)((e / CH) * (int)pe.ldc * 2 + (e % CH) * 16);
      }
      auto store = [&](int m) __attribute__((always_inline)) {
        if (inside) {
#pragma unroll
          for (int it = 0; it < kIt16; ++it)
            __builtin_nontemporal_store(val[it], (u32x4_any_t*)(wave_c + (lane_off[it] + (uint32_t)m * band_step)));
          return;
        }
#pragma unroll
        for (int it = 0; it < kIt16; ++it) {
          const int e = it * 64 + slane;
          const int r = e / CH, q = e % CH;
          const int i = row0 + wm * Cfg::WTM + m * 16 + r;
          const int j = col0 + wn * Cfg::WTN + q * 8;
          if (i < pe.M && j < pe.N) {
            TO* c = Cb + (int64_t)i * pe.ldc + j;
            if (j + 8 <= pe.N) {
              __builtin_nontemporal_store(val[it], (u32x4_any_t*)c);   // C is not read again here: keep it from displacing A and B in L2
            } else {                               // ragged right edge: element by element
#pragma unroll
              for (int t2 = 0; t2 < 8; ++t2) {
                const uint32_t word = val[it][t2 >> 1];
                const uint16_t h = (t2 & 1) ? (uint16_t)(word >> 16) : (uint16_t)(word & 0xffffu);
                if (j + t2 < pe.N) ((uint16_t*)c)[t2] = h;
              }
            }
          }
        }
      };
      values(std::integral_constant<int, 0>());
      static_for<0, MT>([&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value;
        write(m & 1);
        if constexpr (m > 0) read((m - 1) & 1);
        if constexpr (m + 1 < MT) values(std::integral_constant<int, m + 1>());
        if constexpr (m > 0) store(m - 1);
      });
      read((MT - 1) & 1);
      store(MT - 1);
    };
    // fp32 through LDS.  128x128 tiles: half a band at a time (16 rows of half the wave's columns, as many bytes as a 16-bit band),
    // pipelined like those.  What bounds them at a short K is latency: one band at a time, write, wait, read and store in series,
    // 429x6795x256 with fp8 operands took 10.0 us, 9.4 so (bf16 11.9, 11.2), 4096x4096x512 25.6, 23.7; 3357 drawn fp8 and 4396 bf16 products with
    // K up to 2048 0.967.  The larger tiles, whose two waves per SIMD overlap each other's bands: one whole band at a time.  Halves there, whose
    // stores are one line, take up to 1.02 with 30 million and more results in rows off lines; two to four bands before the first store
    // 0.98 on average, but 1.07 for 985x8779x1024 on 256x192 tiles (20.7 us).  Straight from the accumulators, 64 bytes of a row per
    // store: 0.95 with few tiles, up to 1.24 where C is most of the work.
    auto put = [&](f32x4_any_t* c, const f32x4_t& v) __attribute__((always_inline)) {
      if (pe.c_cached) *c = v;                     // split-K partials are read by the next kernel
      else __builtin_nontemporal_store(v, c);
    };
    auto drain32_halves = [&](auto actf) __attribute__((always_inline)) {
      static_assert(NT % 2 == 0, "half bands of whole fragments");
      constexpr int NH = NT / 2;
      float* Cf = (float*)pe.C + (int64_t)batch * pe.stride_c;
      const int slane = fresh_lane();
      f32x4_t w[NH];
      f32x4_t val[kIt16];
      float bvs[NT][4];                           // the bias of this lane's columns, the same for every band
#pragma unroll
      for (int n = 0; n < NT; ++n) bias4(col0 + wn * Cfg::WTN + n * 16 + eq * 4, bvs[n]);
      auto values = [&](auto h_c) __attribute__((always_inline)) {
        constexpr int m = decltype(h_c)::value / 2, n0 = decltype(h_c)::value % 2 * NH;
#pragma unroll
        for (int n = 0; n < NH; ++n)
#pragma unroll
          for (int e = 0; e < 4; ++e) w[n][e] = actf(acc[m][n0 + n][e] + bvs[n0 + n][e]);
      };
      auto write = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NH; ++n) *(f32x4_t*)(wt + buf * kBand16 + er * OROWB + (((n * 4 + eq) ^ osw(er)) * 16)) = w[n];
      };
      auto read = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kIt16; ++it) {
          const int e = it * 64 + slane;
          const int r = e / CH, q = e % CH;
          val[it] = *(const f32x4_t*)(wt + buf * kBand16 + r * OROWB + ((q ^ osw(r)) * 16));
        }
      };
      const bool inside = row0 + BM <= pe.M && col0 + BN <= pe.N && (int64_t)BM * pe.ldc * 4 < ((int64_t)1 << 31);
      char* const wave_c = (char*)(Cf + (int64_t)(row0 + wm * Cfg::WTM) * pe.ldc + col0 + wn * Cfg::WTN);
      const uint32_t band_step = (uint32_t)(16 * pe.ldc * 4);
      uint32_t lane_off[kIt16];
#pragma unroll
      for (int it = 0; it < kIt16; ++it) {
        const int e = it * 64 + slane;
        lane_off[it] = (uint32_t)((e / CH) * (int)pe.ldc * 4 + (e % CH) * 16);
      }
      auto store = [&](int h) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < kIt16; ++it) {
          if (inside) {
            put((f32x4_any_t*)(wave_c + (lane_off[it] + (uint32_t)(h / 2) * band_step + (h % 2) * OROWB)), val[it]);
            continue;
          }
          const int e = it * 64 + slane;
          const int r = e / CH, q = e % CH;
          const int i = row0 + wm * Cfg::WTM + h / 2 * 16 + r;
          const int j = col0 + wn * Cfg::WTN + h % 2 * (NH * 16) + q * 4;
          if (i < pe.M && j < pe.N) {
            float* c = Cf + (int64_t)i * pe.ldc + j;
            if (j + 4 <= pe.N) {
              put((f32x4_any_t*)c, val[it]);
            } else {
#pragma unroll
              for (int t2 = 0; t2 < 4; ++t2)
                if (j + t2 < pe.N) c[t2] = val[it][t2];
            }
          }
        }
      };
      values(std::integral_constant<int, 0>());
      static_for<0, 2 * MT>([&](auto h_c) __attribute__((always_inline)) {
        constexpr int h = decltype(h_c)::value;
        write(h & 1);
        if constexpr (h > 0) read((h - 1) & 1);
        if constexpr (h + 1 < 2 * MT) values(std::integral_constant<int, h + 1>());
        if constexpr (h > 0) store(h - 1);
      });
      read(1);
      store(2 * MT - 1);
    };
    auto drain32_bands = [&](auto actf) __attribute__((always_inline)) {
      float* Cf = (float*)pe.C + (int64_t)batch * pe.stride_c;
      const int slane = fresh_lane();
      constexpr int OROWB32 = Cfg::WTN * 4, CH32 = OROWB32 / 16, kIt32 = 16 * CH32 / 64;   // bytes, pieces per fp32 row of the wave's block
      constexpr int kKey32 = OROWB == 192 ? 7 : 15;          // chunk-slot key, see osw
      static_assert(16 * OROWB32 <= kShare, "one 16-row band of the wave block in fp32 must fit the wave's share of LDS");
      const bool inside = row0 + BM <= pe.M && col0 + BN <= pe.N && (int64_t)BM * pe.ldc * 4 < ((int64_t)1 << 31);
      char* const wave_c = (char*)(Cf + (int64_t)(row0 + wm * Cfg::WTM) * pe.ldc + col0 + wn * Cfg::WTN);
      const uint32_t band_step = (uint32_t)(16 * pe.ldc * 4);
      uint32_t lane_off[kIt32];
#pragma unroll
      for (int it = 0; it < kIt32; ++it) {
        const int e = it * 64 + slane;
        lane_off[it] = (uint32_t)((e / CH32) * (int)pe.ldc * 4 + (e % CH32) * 16);
      }
      static_for<0, MT>([&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          float bv[4];
          bias4(col0 + wn * Cfg::WTN + n * 16 + eq * 4, bv);
          f32x4_t w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = actf(acc[m][n][e] + bv[e]);
          const int q = n * 4 + eq;
          *(f32x4_t*)(wt + er * OROWB32 + ((q ^ (er & kKey32)) * 16)) = w;
        }
#pragma unroll
        for (int it = 0; it < kIt32; ++it) {
          const int e = it * 64 + slane;
          const int r = e / CH32, q = e % CH32;
          const f32x4_t val = *(const f32x4_t*)(wt + r * OROWB32 + ((q ^ (r & kKey32)) * 16));
          if (inside) {
            put((f32x4_any_t*)(wave_c + (lane_off[it] + (uint32_t)m * band_step)), val);
            continue;
          }
          const int i = row0 + wm * Cfg::WTM + m * 16 + r;
          const int j = col0 + wn * Cfg::WTN + q * 4;
          if (i < pe.M && j < pe.N) {
            float* c = Cf + (int64_t)i * pe.ldc + j;
            if (j + 4 <= pe.N) {
              put((f32x4_any_t*)c, val);
            } else {
#pragma unroll
              for (int t2 = 0; t2 < 4; ++t2)
                if (j + t2 < pe.N) c[t2] = val[t2];
            }
          }
        }
      });
    };
    // dest: 1 = 16-bit, 2 = fp32
    auto drain_to = [&](auto actf, auto dest) __attribute__((always_inline)) {
      if constexpr (decltype(dest)::value == 2 && BM * BN <= 128 * 128) drain32_halves(actf);
      else if constexpr (decltype(dest)::value == 2) drain32_bands(actf);
      else drain16_all(actf);
    };
    auto drain_by_activation = [&](auto dest) __attribute__((always_inline)) {
      switch (act) {
        case kActRelu: drain_to([](float x) { return fmaxf(x, 0.0f); }, dest); break;
        case kActGeluErf: drain_to([](float x) { return gelu_erf_f32(x); }, dest); break;
        case kActGeluTanh: drain_to([](float x) { return gelu_tanh_f32(x); }, dest); break;
        case kActSwishScale: { const float c = pe.scale; drain_to([c](float x) { return swish_scale_f32(x, c); }, dest); } break;
        case kActSigmoidScaleResidual: { const float c = pe.scale; drain_to([c](float x) { return sigmoid_scale_residual_f32(x, c); }, dest); } break;
        default: drain_to([](float x) { return x; }, dest); break;
      }
    };

    if constexpr (!PERSIST) {
      __builtin_amdgcn_s_barrier();              // all waves are done reading the slab stages
      asm volatile("" ::: "memory");
    }
    if (pe.c_f32) {
      drain_by_activation(std::integral_constant<int, 2>());
      return;
    }
    drain_by_activation(std::integral_constant<int, 1>());
  };

  // ---- main loop ------------------------------------------------------------------------
  // Slab t lives in LDS stage t % S.  The hand-over to slab t+1 (own reads retired, own loads
  // landed, all waves met) sits before the last sub-step of slab t, whose fragments are
  // already in registers; stage t % S is free from then on and is refilled with slab t+S over
  // the next LW sub-steps (the last one of slab t and, LW > 1, the first ones of slab t+1), which
  // leaves the remaining sub-steps before the next hand-over for the loads to land.  With two stages
  // that is all the time they have, and panels that come from HBM need most of it: the eight-wave tile
  // spreads its loads over two sub-steps (operands outside the last-level cache, 4096x14336x4096: 402 us
  // with three, 371 with two on one box; a single sub-step is 1 % slower again).
  // Priorities (two waves per SIMD): highest right after the hand-over, one lower per
  // sub-step, so the wave that is behind runs first.
  const int T_full = p.K / BK;
  constexpr int LW = Cfg::kWaves == 8 ? 2 : (NSUB >= 4 ? NSUB - 1 : 1);   // sub-steps the loads of a slab are spread over
  int stage = 0, t = 0;
  SlabIo io_none{nullptr, nullptr, 0u, 0u};
  auto next_read_stage = [&]() __attribute__((always_inline)) {      // (S > 2: forward by one, or back to stage 0)
    const int by = stage + 1 == S ? -(S - 1) * Cfg::STAGE_BYTES : Cfg::STAGE_BYTES;
#pragma unroll
    for (int x = 0; x < NA; ++x) a_rd[x] += by;
#pragma unroll
    for (int x = 0; x < NB; ++x) b_rd[x] += by;
  };
  // early: the rest of the loads of slab t+S-1 (begun after the previous hand-over) into the stage before this one, so that
  // the S-2 slabs after the next one are requested and the wait for the next one leaves their loads in flight; late: the first
  // loads of slab t+S into this stage after the hand-over.  (One body for all slabs but the last S, one for those, each in a loop of
  // its own: with copies of the body in the branches of a condition the compiler moved accumulators between registers where
  // the branches met, with none of the wait states that MFMAs in assembly need around such moves.)
  auto slab_body = [&](auto late_c, bool early) __attribute__((always_inline)) {
    constexpr bool late = decltype(late_c)::value;
    const int before = S == 2 ? stage ^ 1 : (stage == 0 ? S - 1 : stage - 1);
    const SlabIo io_early = slab_io(t + S - 1, before), io_late = slab_io(t + S, stage);
    static_for<0, NSUB - 1>([&](auto u_c) __attribute__((always_inline)) {
      constexpr int u = decltype(u_c)::value;
      set_prio(u < 3 ? 2 - u : 0);
      constexpr int q0 = kLoads * (u + 1) / LW, q1 = kLoads * (u + 2) / LW;
      if constexpr (PF && late && u == LW - 1) prefetch(Ab + (int64_t)(t + 2) * a_step, Bb + (int64_t)(t + 2) * b_step);
      if constexpr (u + 1 < LW)
        sub_step(u_c, true, q0 < kLoads ? q0 : kLoads, q1 < kLoads ? q1 : kLoads, io_early, early);
      else
        sub_step(u_c, true, 0, 0, io_none);
    });
    if (early) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * kLoads + (PF && late ? 1 : 0)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    set_prio(3);
    if constexpr (S == 2) flip_read_stage();
    else next_read_stage();
    sub_step(std::integral_constant<int, NSUB - 1>(), true, 0, late ? kLoads / LW : 0, io_late);
    stage = S == 2 ? stage ^ 1 : (stage + 1 == S ? 0 : stage + 1);
  };
  typedef std::integral_constant<bool, true> yes_t;
  typedef std::integral_constant<bool, false> no_t;

  if constexpr (!PERSIST) {
  if constexpr (PRE) {
    if (T_full * BK < p.K) {
#pragma unroll
      for (int q = 0; q < kLoads; ++q) tail_v[q] = load_tail_q(T_full, q);
    }
  }
  if (T_full > 0) {
    // the first S-1 slabs (as many as there are) and the first part of the next; the first one has landed when the others'
    // loads are left
    static_for<0, S>([&](auto q_c) __attribute__((always_inline)) {
      constexpr int sl = decltype(q_c)::value;
      if (sl < T_full) {
        const SlabIo io = slab_io(sl, sl);
#pragma unroll
        for (int q = 0; q < (sl == S - 1 ? kLoads / LW : kLoads); ++q) issue_one_load(q, io);
      }
    });
    if (T_full >= S) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * kLoads + kLoads / LW) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_all(std::integral_constant<int, 0>());
  }
  for (t = 0; t < T_full - S; ++t) slab_body(yes_t(), true);
  for (; t < T_full; ++t) slab_body(no_t(), t + S <= T_full);
  set_prio(0);
  // the last fragment reads (of a stage nobody multiplies) are still in flight
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  if (stage) set_read_stage(0, lane);          // the K tail reads stage 0
  if (T_full * BK < p.K) {                     // K tail, through registers with zero fill
    __builtin_amdgcn_s_barrier();              // every wave is done with the LDS stages
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      if constexpr (!PRE) tail_v[q] = load_tail_q(T_full, q);
      store_tail_q(q, tail_v[q]);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int ksteps = (p.K - T_full * BK + Frag16<T>::kStep - 1) / Frag16<T>::kStep;
    static_for<0, NSUB>([&](auto u_c) __attribute__((always_inline)) {
      constexpr int u = decltype(u_c)::value;
      if (u / G < ksteps) {
        read_all(u_c);
        sub_step(u_c, false, 0, 0, io_none);
      }
    });
    wait_lgkmcnt<0>();
  }
  batch = ld_batch;
  epilogue(ld_tm * BM, ld_tn * BN);
  } else {
  // ---- persistent: the tiles of this workgroup as one stream of slabs ------------------------
  // The loads run two slabs ahead of the MFMAs and simply carry on into the next tile's panels:
  // every slab body but the last two of the last tile requests loads.  ld_a / ld_b and the lane
  // offsets describe the slab the loads are at; they move on one slab at a time and switch to
  // the next tile when this one's slabs are all requested.
  int ld_vid = blockIdx.x, ld_t = 0;
  int cur_tm = ld_tm, cur_tn = ld_tn, cur_batch = ld_batch;     // the tile being multiplied
  auto fresh_lane_id = []() __attribute__((always_inline)) {
    unsigned z = 0;
    asm volatile("" : "+v"(z));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, z));
  };
  auto next_slab = [&]() __attribute__((always_inline)) {
    ld_a += a_step; ld_b += b_step;
    if (++ld_t == T_full) {
      ld_t = 0;
      ld_vid += gridDim.x;
      if (ld_vid < total_tiles) {
        const MfmaArgs q = tile_args();
        locate(q, ld_vid);
        load_tile(q, fresh_lane_id(), 0);        // (no lane id kept in a register across the loop)
      }
    }
  };
  // tile_end (compile time): the last slab of a tile; its last sub-step requests no fragments (the
  // next tile's first ones are read after the epilogue, which then has no fragment registers to
  // keep alive).  touch (compile time): whether a slab of this tile is left to prefetch: in all but the
  // last two (the loads of the last one are under way by then; touching it again cost 64 x (512x512x128),
  // two slabs, 0.1 us of 12).  early / late (run time; true in every slab but the last two of the last tile):
  // whether the rest of one slab's loads and the first part of the next one's are requested.
  auto body = [&](auto touch_c, auto end_c, bool early, bool late) __attribute__((always_inline)) {
    constexpr bool touch = PF && decltype(touch_c)::value, tile_end = decltype(end_c)::value;
    const SlabIo io_early = slab_io_at(ld_a, ld_b, stage ^ 1);
    static_for<0, NSUB - 1>([&](auto u_c) __attribute__((always_inline)) {
      constexpr int u = decltype(u_c)::value;
      set_prio(u < 3 ? 2 - u : 0);
      constexpr int q0 = kLoads * (u + 1) / LW, q1 = kLoads * (u + 2) / LW;
      if constexpr (touch && u == LW - 1) prefetch(ld_a + a_step, ld_b + b_step);
      if constexpr (u + 1 < LW)
        sub_step(u_c, true, q0 < kLoads ? q0 : kLoads, q1 < kLoads ? q1 : kLoads, io_early, early);
      else
        sub_step(u_c, true, 0, 0, io_none);
    });
    if (late) next_slab();                     // the early part was the rest of a slab: on to the next one
    const SlabIo io_late = slab_io_at(ld_a, ld_b, stage);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(touch ? 1 : 0) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    set_prio(3);
    flip_read_stage();
    sub_step(std::integral_constant<int, NSUB - 1>(), !tile_end, 0, kLoads / LW, io_late, late);
    stage ^= 1;
  };
  // slab 0 whole and the first part of slab 1; from then on every body requests the rest of one
  // slab and the first part of the next
  {
    const SlabIo io0 = slab_io_at(ld_a, ld_b, 0);
#pragma unroll
    for (int q = 0; q < kLoads; ++q) issue_one_load(q, io0);
    next_slab();
    const SlabIo io1 = slab_io_at(ld_a, ld_b, 1);
#pragma unroll
    for (int q = 0; q < kLoads / LW; ++q) issue_one_load(q, io1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads / LW) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
  for (int vid = blockIdx.x; vid < total_tiles; vid += gridDim.x) {
    const bool last = vid + (int)gridDim.x >= total_tiles;
    read_all(std::integral_constant<int, 0>());
    for (t = 0; t < T_full - 2; ++t) body(yes_t(), no_t(), true, true);
    body(no_t(), no_t(), true, !last);
    body(no_t(), yes_t(), !last, !last);
    set_prio(0);
    wait_lgkmcnt<0>();
    batch = cur_batch;
    epilogue(cur_tm * BM, cur_tn * BN);
    cur_tm = ld_tm; cur_tn = ld_tn; cur_batch = ld_batch;     // (the loads are in the next tile by now)
    if (!last) {
      // the lane-dependent offsets and addresses are derived afresh here (from an opaque copy of the
      // lane id, so that the compiler cannot keep the earlier ones alive across the epilogue instead)
      const int lane_now = fresh_lane_id();
      load_tile(tile_args(), lane_now, ld_t);
      set_read_stage(stage, lane_now);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[m][n][r] = 0.0f;
      // (the next MFMAs are assembly statements the compiler's hazard recogniser cannot see: give the
      // accumulator writes above time to retire, and keep them above this point)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) asm volatile("" : "+a"(acc[m][n]));
      asm volatile("s_nop 7" ::: "memory");
    }
  }
  }
}

}  // namespace mi355gemm
