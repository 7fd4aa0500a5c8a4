// Join GEMM of the HOTRG block-spin contraction on gfx950 MFMA.
//
// C[m][n] (+)= sum_k A[m][k] * Bt[n][k]: both operands K-contiguous, so a
// workgroup streams BM rows of A and BN rows of Bt through LDS in tiles of
// RB bytes of K per row.  Inside a tile, lane group g = lane/16 of a wave
// owns bytes [g RB/4, (g+1) RB/4) of every row it reads; the k values a lane
// feeds to successive MFMAs are therefore contiguous in LDS, and A and B use
// the same assignment, so the contraction over k is unchanged.
//
//   FP64   v_mfma_f64_16x16x4_f64   gemm_pipe_kernel: 128 x 128, 64 x 128 or
//          64 x 64 tile by four waves, RB 128 (16 doubles, 4 MFMA k-steps);
//          gemm_ksplit_kernel where the 64 x 64 tiles do not fill the chip
//   FP32   v_mfma_f32_16x16x4_f32   gemm_pipe_kernel: 64 x 128 or 64 x 64 tile,
//          RB 128 (32 floats, 8 k-steps); the MFMA sums 4 K tiles (128
//          products) in FP32, the groups are summed in FP64
//   BF16X3 v_mfma_f32_16x16x32_bf16 gemm_split_kernel, two planes: 256 x 256
//          tile of eight 128 x 64 waves or 128 x 128 of four 64 x 64; three
//          products hi*hi + hi*lo + lo*hi into one FP32 accumulator
//   BF16X6 the same kernel, three planes (fl32(a) = hi + mid + lo exactly): 128
//          x 128 tile of eight 64 x 32 waves or 64 x 64 of four 32 x 32; six
//          products hi*hi + hi*mid + mid*hi + mid*mid + hi*lo + lo*hi; the
//          MFMA sums BF6_FLUSH K tiles in FP32, the groups are summed in
//          FP64 (FP32-accurate operands and FP64-grade accumulation)
//
// Workgroup ids are remapped (ids are dealt round-robin to the 8 XCDs).  FP64
// and FP32: each XCD works on one contiguous range of tiles, walked in groups of
// GROUP_M tile-rows, so that neighbouring tiles on one XCD share A and Bt rows
// in that XCD's L2.  Split BF16: the XCDs also share blocks (tile_coords_shared).
// In FP64 that order is 0.3 % slower; in FP32 it gives 7808^2 x 7776 132.9 against
// 130.5 TFLOP/s and 8192^2 x 8192 137.8 against 138.4.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace trg {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // at any bf16 element

// FP32 join: K tiles (32 floats each) summed by the MFMA in FP32 before the
// partial sum is added to the FP64 accumulator
constexpr uint32_t F32_FLUSH = 4;
constexpr int GROUP_M = 8;

// BF16X6 join: K tiles (32 elements each) per FP32 group
constexpr int BF6_FLUSH = 4;

template <int PREC> struct Prec;
template <> struct Prec<0> {  // FP64
  using in_t = double;
  using out_t = double;
  using acc_t = v4d;
  using frag_t = d2;
  static constexpr int planes = 1;
  static constexpr int elem = 8;
};
template <> struct Prec<1> {  // FP32
  using in_t = float;
  using out_t = float;
  using acc_t = v4f;
  using frag_t = f4;
  static constexpr int planes = 1;
  static constexpr int elem = 4;
};
template <> struct Prec<2> {  // BF16 x3
  using in_t = uint16_t;
  using out_t = float;
  using acc_t = v4f;
  using frag_t = bf16x8;
  static constexpr int planes = 2;
  static constexpr int elem = 2;
};
template <> struct Prec<3> {  // BF16 x6
  using in_t = uint16_t;
  using out_t = float;
  using acc_t = v4f;
  using frag_t = bf16x8;
  static constexpr int planes = 3;
  static constexpr int elem = 2;
};

__device__ inline void tile_coords(uint32_t wg, uint32_t tiles_m, uint32_t tiles_n, uint32_t &tm,
                                   uint32_t &tn) {
  const uint32_t total = tiles_m * tiles_n;
  // XCD-contiguous renumbering (bijective for any total)
  const uint32_t xcd = wg % NUM_XCD, idx = wg / NUM_XCD;
  const uint32_t per = total / NUM_XCD, rem = total % NUM_XCD;
  const uint32_t w = xcd * per + (xcd < rem ? xcd : rem) + idx;
  // grouped raster: GROUP_M tile-rows walked column by column
  const uint32_t group_size = GROUP_M * tiles_n;
  const uint32_t group = w / group_size;
  const uint32_t first_m = group * GROUP_M;
  const uint32_t gm = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
  const uint32_t in_group = w % group_size;
  tm = first_m + in_group % gm;
  tn = in_group / gm;
}

// Tiles of the split-BF16 kernels.  The large ones run one workgroup per CU, so
// 256 in a round, laid out as 16 x 16 tiles of which each XCD takes 8 x 4 (the
// small ones, several per CU and few rounds, keep the order).  Its L2 serves the 12
// panels of those as before, and the 8 XCDs together stream 32 panels instead
// of 96, so that most of what one XCD misses another has just brought into the
// memory-side cache.  Bijective for any grid: blocks of 256 workgroups are
// consecutive in the raster (the last, smaller one cut evenly among the XCDs),
// which walks row groups of 16 in strips of 4 columns, each strip's upper 8
// rows first.
// Measured against each XCD walking its own eighth of the tiles in groups of 4
// (BF16x6) or 8 rows (BF16x3), TFLOP/s: a full slice of the Dcut 10 step, 30080 x
// 100096 x 100000, 179.5 -> 205.6 (6.6 -> 5.5 TB read from beyond the L2s, MFMA
// pipes 47 -> 52 % busy at 2.26 and 2.27 GHz); 10112 x 10112 x 100000 random
// operands 178 -> 188 (pipes 56 % busy at 1.79 -> 1.88 GHz, where the power limit
// sets the clock); BF16x3 13312 x 13312 x 59072 469 -> 490 (1.60 -> 1.66 GHz).
__device__ inline void tile_coords_shared(uint32_t wg, uint32_t tiles_m, uint32_t tiles_n, uint32_t &tm, uint32_t &tn) {
  constexpr uint32_t ROUND = 256, GM = 16, SW = 4, HALF = 8;
  const uint32_t total = tiles_m * tiles_n, base = wg / ROUND * ROUND;
  const uint32_t n = total - base < ROUND ? total - base : ROUND;
  const uint32_t xcd = wg % NUM_XCD, idx = (wg - base) / NUM_XCD;
  const uint32_t per = n / NUM_XCD, rem = n % NUM_XCD;
  const uint32_t w = base + xcd * per + (xcd < rem ? xcd : rem) + idx;
  const uint32_t first_m = w / (GM * tiles_n) * GM;
  const uint32_t gm = tiles_m - first_m < GM ? tiles_m - first_m : GM;
  const uint32_t in_group = w - first_m * tiles_n;
  const uint32_t strip = in_group / (gm * SW), i = in_group % (gm * SW);
  const uint32_t sw = tiles_n - strip * SW < SW ? tiles_n - strip * SW : SW;
  const bool split = gm == GM;
  const uint32_t rows = split ? HALF : gm;
  const uint32_t half = split ? i / (HALF * sw) : 0;
  const uint32_t j = i - half * HALF * sw;
  tm = first_m + half * HALF + j % rows;
  tn = strip * SW + j / rows;
}

// ------------------------------------------------ pipelined FP64 / FP32 join ---
// LDS layout of the pipelined kernel: rows of 128 bytes (8 chunks of 16),
// two rows per 256-byte line; chunk c of row r sits at chunk c ^ pipe_swz(r).
// A 16-byte read of a wave runs in four phases; the 16 lanes of one phase
// hold eight rows of each parity, four of them one lane group (two chunks)
// further on, so pipe_swz takes odd values on rows 0-3 and 12-15 and even
// ones on rows 4-11 (mod 16): all 16 land on different 4-bank groups.
__device__ inline int pipe_swz(int row) {
  return int((0x75642031u >> (4 * ((row >> 1) & 7))) & 7u);
}

// C (+)= A Bt^T for one BM x BN tile by WM x WN waves, K in tiles of 128
// bytes per row.  Bound by the MFMA issue rate (64 cycles per FP64 and 32 per
// FP32 MFMA), so the design keeps every other instruction behind an MFMA: both
// halves of a K tile's fragments live in registers, and while the MFMAs of one
// half run, the other half (or the first half of the next tile) is read from
// LDS, the next tile is stored to the other LDS stage and the one after that
// is loaded from memory; the barrier of a tile falls between two MFMA groups.
// MINW waves per SIMD come from different workgroups, so one workgroup's
// barrier is covered by another's MFMAs.  The FP32 64 x 128 tile, with FP64
// sums beside its accumulators, does not fit the 256 registers that two waves
// per SIMD leave: 76 spill (172 bytes of scratch per lane).
//
// Measured (M = N = 10112, K = 25008 / 25056): FP64 58.3 -> 72.3 TFLOP/s (92 %
// of 78.6; MFMA pipes busy 77 -> 96 % at 8192^2), FP32 96 -> 138 TFLOP/s
// (88 % of 157; busy 70 -> 91 %), against a kernel that read all fragments of a
// tile from LDS right before its MFMAs with one wave per SIMD (FP64) or two in
// step (FP32).  Of the FP32 gain, 129 -> 138 comes from adding a finished
// group to the FP64 sums block by block between the next tile's first MFMAs.
//
// RIGHT selects the right operand: RowsRight is the K-contiguous Bt above;
// ColsRight (FP64 only) reads B as it lies in memory with its columns
// contiguous, element (k, n) at (k / k1) sk2 + (k % k1) sk1 + (n / n1) sn2 + n % n1,
// so that a tensor whose summed leg is an outer one needs no transposed copy.
// A K tile of it is 16 rows of BN columns; its LDS rows are BN + 4 doubles, so
// the two rows of a half wave's 8-byte reads fall on different banks.  Rows
// past K repeat the last one (A is zero there), columns past N the last one
// (not stored); C is M x N, unpadded.
// Measured: 13824 x 2880 x 576 in 128 x 128 tiles 62 TFLOP/s, 576 x 2880 x
// 13824 in six K ranges of 64 x 128 tiles 61, as fast as from packed
// operands (63 and 61), whose copies took half as long again.
struct RowsRight {
  static constexpr bool cols = false, pairs = false;
};
template <bool PAIRS>   // columns 2 i and 2 i + 1 adjacent and 16-byte aligned
struct ColsRight {
  static constexpr bool cols = true, pairs = PAIRS;
  uint32_t M, N, K, k1, n1;
  uint64_t sk1, sk2, sn2;
};

template <int PREC, int BM, int BN, int WM, int WN, int MINW, bool ACCUM, class RIGHT = RowsRight>
__global__ void __launch_bounds__(64 * WM * WN, MINW)
gemm_pipe_kernel(const typename Prec<PREC>::in_t *__restrict__ A, const typename Prec<PREC>::in_t *__restrict__ Bt,
                 typename Prec<PREC>::out_t *__restrict__ C, uint32_t tiles_m, uint32_t tiles_n, uint32_t ktiles,
                 uint64_t lda, uint64_t ldb, uint64_t ldc, uint64_t c_split_stride, uint64_t batch_a,
                 uint64_t batch_b, uint64_t batch_c, RIGHT rt) {
  using P = Prec<PREC>;
  using acc_t = typename P::acc_t;
  using frag_t = typename P::frag_t;
  constexpr bool COLS = RIGHT::cols;
  static_assert(!COLS || PREC == 0, "column-contiguous right operands are FP64");
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 16, FN = TN / 16;
  constexpr int RB = 128, CPR = 8, BK = RB / P::elem;
  constexpr int LA = BM * CPR / NT, LB = BN * CPR / NT;
  static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads mismatch");
  constexpr int LDN = (BN + 4) * 8;   // bytes of an LDS row of a column-contiguous tile
  constexpr int STAGE = BM * RB + (COLS ? BK * LDN : BN * RB);
  constexpr bool F64SUM = PREC == 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int g = lane >> 4, r16 = lane & 15;
  uint32_t tm, tn;
  tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const uint64_t m0 = uint64_t(tm) * BM, n0 = uint64_t(tn) * BN;
  A += uint64_t(blockIdx.z) * batch_a;
  Bt += uint64_t(blockIdx.z) * batch_b;
  C += uint64_t(blockIdx.z) * batch_c + uint64_t(blockIdx.y) * c_split_stride;
  const uint64_t koff = uint64_t(blockIdx.y) * ktiles * BK;
  const int row0 = tid / CPR, col0 = tid % CPR;   // chunk i of this thread: row row0 + i NT / 8
  const unsigned char *gA = reinterpret_cast<const unsigned char *>(A + (m0 + row0) * lda + koff) + col0 * 16;
  const unsigned char *gB = reinterpret_cast<const unsigned char *>(Bt + (n0 + row0) * ldb + koff) + col0 * 16;
  const uint64_t stepA = uint64_t(NT / CPR) * lda * P::elem, stepB = uint64_t(NT / CPR) * ldb * P::elem;

  // column-contiguous right operand: this thread's pair of columns and its
  // LB rows of a K tile, as (k / k1, k % k1), which advance by 16 a tile
  constexpr int CPT = COLS ? BN / 2 : 1, RSTEP = COLS ? NT / CPT : 1;
  uint32_t ktn = ktiles, kq[COLS ? LB : 1], kr[COLS ? LB : 1];
  uint32_t kleft = 0, kq16 = 0, kr16 = 0, brow = 0, bcol = 0;
  const double *bc0 = nullptr, *bc1 = nullptr;
  uint64_t klast = 0;
  if constexpr (COLS) {
    const uint32_t k0 = uint32_t(koff), total = (rt.K + BK - 1) / BK - blockIdx.y * ktiles;
    ktn = ktiles < total ? ktiles : total;
    brow = uint32_t(tid) / CPT;
    if constexpr (CPT == 64) brow = __builtin_amdgcn_readfirstlane(brow);
    bcol = uint32_t(tid) % CPT * 2;
    // a whole pair stays inside: N is even where pairs are loaded
    const uint32_t c0 = uint32_t(n0) + bcol < rt.N ? uint32_t(n0) + bcol : rt.N - (RIGHT::pairs ? 2 : 1);
    const uint32_t c1 = c0 + 1 < rt.N ? c0 + 1 : rt.N - 1;
    bc0 = Bt + (c0 / rt.n1) * rt.sn2 + c0 % rt.n1;
    bc1 = Bt + (c1 / rt.n1) * rt.sn2 + c1 % rt.n1;
    kq16 = BK / rt.k1;
    kr16 = BK % rt.k1;
    kleft = rt.K - k0;   // rows of this workgroup's first tile and after
    klast = uint64_t((rt.K - 1) / rt.k1) * rt.sk2 + uint64_t((rt.K - 1) % rt.k1) * rt.sk1;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const uint32_t k = k0 + brow + i * RSTEP;
      kq[i] = k / rt.k1;
      kr[i] = k % rt.k1;
    }
  }
  u32x4 ra[LA], rb[LB];
  auto gload = [&](uint32_t kt) {
    const uint64_t kb = uint64_t(kt) * RB;
#pragma unroll
    for (int i = 0; i < LA; ++i) ra[i] = *reinterpret_cast<const u32x4 *>(gA + i * stepA + kb);
    if constexpr (COLS) {
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        uint64_t off = kq[i] * rt.sk2 + kr[i] * rt.sk1;
        off = kt * BK + brow + i * RSTEP < kleft ? off : klast;
        if constexpr (RIGHT::pairs) {
          rb[i] = *reinterpret_cast<const u32x4 *>(bc0 + off);
        } else {
          rb[i] = __builtin_bit_cast(u32x4, frag_t{bc0[off], bc1[off]});
        }
        kq[i] += kq16;
        kr[i] += kr16;
        if (kr[i] >= rt.k1) {
          kr[i] -= rt.k1;
          ++kq[i];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < LB; ++i) rb[i] = *reinterpret_cast<const u32x4 *>(gB + i * stepB + kb);
    }
  };
  // rows of one thread differ by NT / 8, a multiple of 16: one swizzle for all
  static_assert((NT / CPR) % 16 == 0, "swizzle period");
  unsigned char *const sbase = smem + row0 * RB + ((col0 ^ pipe_swz(row0)) << 4);
  auto sstore = [&](int stage) {
#pragma unroll
    for (int i = 0; i < LA; ++i) *reinterpret_cast<u32x4 *>(sbase + stage * STAGE + i * (NT / CPR) * RB) = ra[i];
    if constexpr (COLS) {
#pragma unroll
      for (int i = 0; i < LB; ++i)
        *reinterpret_cast<u32x4 *>(smem + stage * STAGE + BM * RB + (brow + i * RSTEP) * LDN + bcol * 8) = rb[i];
    } else {
#pragma unroll
      for (int i = 0; i < LB; ++i)
        *reinterpret_cast<u32x4 *>(sbase + stage * STAGE + BM * RB + i * (NT / CPR) * RB) = rb[i];
    }
  };
  // half f of a lane's K share of a row: chunk 2 g + f
  const int swz = pipe_swz(r16);
  const int fro[2] = {((2 * g) ^ swz) << 4, ((2 * g + 1) ^ swz) << 4};
  const int abase = (wm * TM + r16) * RB;
  const int bbase = BM * RB + (COLS ? 4 * g * LDN + (wn * TN + r16) * 8 : (wn * TN + r16) * RB);
  frag_t fa[2][FM], fb[2][FN];
  auto fload = [&](int stage, auto half) {
    constexpr int f = decltype(half)::value;
    const unsigned char *s = smem + stage * STAGE + fro[f];
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[f][i] = *reinterpret_cast<const frag_t *>(s + abase + i * 16 * RB);
    if constexpr (COLS) {   // rows 4 g + 2 f and 4 g + 2 f + 1 of the tile
      const unsigned char *sb = smem + stage * STAGE + bbase + 2 * f * LDN;
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) fb[f][j][s2] = *reinterpret_cast<const double *>(sb + s2 * LDN + j * 16 * 8);
    } else {
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[f][j] = *reinterpret_cast<const frag_t *>(s + bbase + j * 16 * RB);
    }
  };
  acc_t acc[FM][FN];
  v4d acc64[F64SUM ? FM : 1][F64SUM ? FN : 1];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      acc[i][j] = acc_t{};
      if constexpr (F64SUM) acc64[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    }
  // k-steps [s0, s1) of half f
  constexpr int KS = 16 / P::elem;   // k-steps of one 16-byte fragment
  auto mfma = [&](auto half, auto first, auto last, auto fold) {
    constexpr int f = decltype(half)::value;
#pragma unroll
    for (int s = decltype(first)::value; s < decltype(last)::value; ++s)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          if constexpr (decltype(fold)::value) {
            if (s == 0) {
#pragma unroll
              for (int e = 0; e < 4; ++e) acc64[i][j][e] += double(acc[i][j][e]);
              acc[i][j] = acc_t{};
            }
          }
          if constexpr (PREC == 0)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[f][i][s], fb[f][j][s], acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[f][i][s], fb[f][j][s], acc[i][j], 0, 0, 0);
        }
  };
  constexpr auto I0 = std::integral_constant<int, 0>{};
  constexpr auto I1 = std::integral_constant<int, 1>{};
  constexpr auto IH = std::integral_constant<int, KS / 2>{};
  constexpr auto IK = std::integral_constant<int, KS>{};
  auto barrier = [&] {   // LDS only: the global loads stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  auto phase = [] { __builtin_amdgcn_sched_barrier(0); };
  // issue order inside a phase: one LDS read per MFMA; one LDS store, one
  // MFMA, one global load, one MFMA
  auto mix_reads = [] {
#pragma unroll
    for (int i = 0; i < FM + FN; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  };
  auto mix_stores = [] {
#pragma unroll
    for (int i = 0; i < LA + LB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  };

  gload(0);
  sstore(0);
  if (ktn > 1) gload(1);
  barrier();
  fload(0, I0);
  // one K tile: `store`: tile kt + 1 (in registers) goes to the other stage, `load`: tile kt + 2 is fetched
  auto body = [&](uint32_t kt, auto fold, auto store, auto load) {
    constexpr bool ST = decltype(store)::value, LD = decltype(load)::value;
    constexpr auto NF = std::false_type{};
    const int cur = kt & 1;
    fload(cur, I1);
    mfma(I0, I0, IH, fold);
    if constexpr (!decltype(fold)::value) mix_reads();
    phase();
    if constexpr (ST) sstore(cur ^ 1);
    if constexpr (LD) gload(kt + 2);
    mfma(I0, IH, IK, NF);
    if constexpr (ST) mix_stores();
    phase();
    barrier();
    if constexpr (ST) fload(cur ^ 1, I0);
    mfma(I1, I0, IK, NF);
    if constexpr (ST) mix_reads();
    phase();
  };
  constexpr auto YES = std::true_type{};
  constexpr auto NO = std::false_type{};
  uint32_t kt = 0;
  if constexpr (F64SUM) {
    auto tail = [&](uint32_t k, auto st, auto ld) {
      if (k % F32_FLUSH == 0) body(k, YES, st, ld);
      else body(k, NO, st, ld);
    };
    for (; kt + F32_FLUSH + 1 < ktiles; kt += F32_FLUSH) {
      body(kt, YES, YES, YES);
#pragma unroll
      for (uint32_t u = 1; u < F32_FLUSH; ++u) body(kt + u, NO, YES, YES);
    }
    while (kt + 2 < ktiles) tail(kt++, YES, YES);
    if (kt + 1 < ktiles) tail(kt++, YES, NO);
    tail(kt, NO, NO);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc64[i][j][e] += double(acc[i][j][e]);
  } else {
    while (kt + 2 < ktn) body(kt++, NO, YES, YES);
    if (kt + 1 < ktn) body(kt++, NO, YES, NO);
    body(kt, NO, NO, NO);
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // row of accumulator e: 4 g + e for the FP32 instruction, g + 4 e for the FP64 one
        const int row = PREC == 0 ? g + 4 * e : 4 * g + e;
        if constexpr (COLS) {
          if (m0 + wm * TM + i * 16 + row >= rt.M || n0 + wn * TN + j * 16 + r16 >= rt.N) continue;
        }
        auto *dst = C + (m0 + wm * TM + i * 16 + row) * ldc + n0 + wn * TN + j * 16 + r16;
        if constexpr (F64SUM)
          *dst = ACCUM ? float(double(*dst) + acc64[i][j][e]) : float(acc64[i][j][e]);
        else
          *dst = ACCUM ? *dst + acc[i][j][e] : acc[i][j][e];
      }
}

// ------------------------------------------------------ split-BF16 joins ---
// 16 bytes per lane from memory straight into LDS: lane l's go to lds + 16 l
// (lds: wave-uniform byte offset).  No register receives the data; the
// compiler does not count the load, so wait_vm must cover it before a barrier
// publishes it.  Writing M0 needs one wait state before the load reads it.
// M0 is reserved: the compiler takes no clobber of it and writes it itself
// right before each instruction that reads it, of which these kernels have none.
__device__ inline void dma16(const void *p, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(lds) : "memory");
}
template <int N>
__device__ inline void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Chunk swizzle of 64-byte LDS rows (four chunks of 16 bytes, four rows per
// 256-byte line): chunk c of row r sits at chunk c ^ split_swz(r).  The 16
// lanes of one phase of a 16-byte read hold rows 0-3 and 12-15 of one chunk
// and rows 4-11 of the next: 0, 2, 3, 1 over r / 4 puts them on 16 different
// 4-bank groups (r / 4 itself does not: 37 % of the LDS cycles were conflicts).
__device__ inline int split_swz(int row) { return int((0x1320u >> (4 * ((row >> 2) & 3))) & 3u); }

// The split-BF16 joins: PL planes per operand (2: hi*hi + hi*lo + lo*hi; 3:
// the six products down to 2^-24), K in tiles of 32 elements (64-byte rows),
// small products first.
//
// What bounds it: an MFMA takes 16 cycles, so a K tile is over in 1536 (PL 3,
// 128 x 128) to 3072 cycles (PL 2, 256 x 256) and neither LDS reads nor the
// 1-2 us of a load from beyond L2 may stand between two tiles.  On dense
// operands the power limit holds the clock at 1.7-1.9 GHz (of 2.4), with the
// pipes 56 to 80 % busy.  Hence:
// - tiles go from memory straight to LDS (no staging registers, no LDS
//   stores), issued NST tiles ahead into a ring of NST stages;
// - every LDS read is issued half a tile ahead of the MFMAs that use it, A in
//   halves of the wave's rows, B in two register sets;
// - reads and loads are issued one by one between MFMAs (issued in a block,
//   the loads of all waves queue in front of the MFMAs);
// - one barrier per tile, between the two halves.
// PL 3: the MFMAs sum FLUSH tiles in FP32; a finished group is added to FP64
// sums between the first MFMAs of the next one.
//
// DMA false serves operands that do not start on 16 bytes, which loads straight
// to LDS are not known to take: a tile travels through registers.  In the first
// half of a tile the next one is stored to LDS (two stages) block by block between
// the MFMAs, each block's register right away loaded with the tile after that.
// Same products in the same order.  Bound by the second 64 bytes that most rows
// of a tile touch, hence tiles as large as the registers allow.  Operands 2 and 8
// bytes off, TFLOP/s: BF16x6 10112^2 x 25056 125 and 141, BF16x3 10240^2 x 25056 246
// and 277 (188 and 431 aligned), against 101 and 115, 212 and 267 with the stores
// in a block before the barrier, 128 x 128 tiles and the loads of a tile moved by
// the compiler behind the MFMAs that should cover them.
//
// Measured against the kernel before (loads through registers, all fragments
// of a tile read right before its MFMAs), TFLOP/s of the product:
//   PL 3  10112^2 x 25056: 154 -> 178 (1.07 PFLOP/s of MFMA, pipes busy 46 ->
//         57 %); 3200^2 x 3136: 158 -> 192
//   PL 2  10240^2 x 25056: 346 -> 407 (1.22 PFLOP/s); 2048^2 x 8192: 125 -> 338
template <int PL, int BM, int BN, int WM, int WN, int NST, int FLUSH, bool DMA, bool ACCUM>
__global__ void __launch_bounds__(64 * WM * WN)
gemm_split_kernel(const uint16_t *__restrict__ A, const uint16_t *__restrict__ Bt, float *__restrict__ C,
                  uint32_t tiles_m, uint32_t tiles_n, uint32_t ktiles, uint64_t lda, uint64_t ldb, uint64_t ldc,
                  uint64_t planeA, uint64_t planeB, uint64_t batch_a, uint64_t batch_b, uint64_t batch_c) {
  constexpr int NW = WM * WN, TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16, RB = 64;
  constexpr int HM = FM / 2;
  constexpr int LA = BM / 16 / NW, LB = BN / 16 / NW;   // 1 KB blocks (16 rows) per wave and plane
  static_assert(LA >= 1 && LB >= 1, "every wave loads whole blocks");
  static_assert(FLUSH == 0 || FLUSH == 4, "the loop below folds every fourth tile");
  static_assert(DMA || NST == 2, "through registers only with two stages");
  constexpr int PLANE = (BM + BN) * RB, STAGE = PLANE * PL;
  constexpr int PERT = PL * (LA + LB);                  // loads of a wave per tile
  constexpr int NTERM = PL == 3 ? 6 : 3;
  // planes of each product: lo*hi, hi*lo, mid*mid, mid*hi, hi*mid, hi*hi or lo*hi, hi*lo, hi*hi
  constexpr int TA[6] = {PL == 3 ? 2 : 1, 0, PL == 3 ? 1 : 0, 1, 0, 0};
  constexpr int TB[6] = {0, PL == 3 ? 2 : 1, PL == 3 ? 1 : 0, 0, 1, 0};
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN, g = lane >> 4, r16 = lane & 15;
  uint32_t tm, tn;
  tile_coords_shared(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const uint64_t m0 = uint64_t(tm) * BM, n0 = uint64_t(tn) * BN;
  A += uint64_t(blockIdx.z) * batch_a;
  Bt += uint64_t(blockIdx.z) * batch_b;
  C += uint64_t(blockIdx.z) * batch_c;
  // block u of this wave: rows 16 (wave LA + u) .. + 15; lane l fills chunk l % 4 of row l / 4
  const int drow = lane >> 2, dchunk = (lane & 3) ^ split_swz(drow);
  const unsigned char *pa[PL][LA], *pb[PL][LB];
#pragma unroll
  for (int p = 0; p < PL; ++p) {
#pragma unroll
    for (int u = 0; u < LA; ++u)
      pa[p][u] = reinterpret_cast<const unsigned char *>(A + p * planeA + (m0 + (wave * LA + u) * 16 + drow) * lda) +
                 dchunk * 16;
#pragma unroll
    for (int u = 0; u < LB; ++u)
      pb[p][u] = reinterpret_cast<const unsigned char *>(Bt + p * planeB + (n0 + (wave * LB + u) * 16 + drow) * ldb) +
                 dchunk * 16;
  }
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(smem));   // low 32 bits of a flat LDS address are its offset
  // one of the PERT blocks of tile kt
  auto dma1 = [&](uint64_t kb, uint32_t base, int q) {
    const int p = q / (LA + LB), u = q % (LA + LB);
    if (u < LA) dma16(pa[p][u] + kb, base + p * PLANE + (wave * LA + u) * 1024);
    else dma16(pb[p][u - LA] + kb, base + p * PLANE + BM * RB + (wave * LB + u - LA) * 1024);
  };
  auto dma = [&](uint32_t kt, uint32_t stage) {
#pragma unroll
    for (int q = 0; q < PERT; ++q) dma1(uint64_t(kt) * RB, lds0 + stage * STAGE, q);
  };
  // the same block into a register, and from there into a stage
  u32x4 rg[DMA ? 1 : PERT];
  auto fetch1 = [&](uint64_t kb, int q) {
    const int p = q / (LA + LB), u = q % (LA + LB);
    rg[q] = *reinterpret_cast<const u32x4_any *>((u < LA ? pa[p][u] : pb[p][u - LA]) + kb);
  };
  auto put1 = [&](uint32_t stage, int q) {
    const int p = q / (LA + LB), u = q % (LA + LB);
    const int at = p * PLANE + (u < LA ? (wave * LA + u) * 1024 : BM * RB + (wave * LB + u - LA) * 1024);
    *reinterpret_cast<u32x4 *>(smem + stage * STAGE + at + lane * 16) = rg[q];
  };
  const int fro = (g ^ split_swz(r16)) << 4;
  const int aoff = (wm * TM + r16) * RB + fro, boff = BM * RB + (wn * TN + r16) * RB + fro;
  bf16x8 fa[PL][FM], fb[2][PL][FN];
  // fragment reads one at a time: q-th of the rows [lo, hi) of A; q-th of B
  auto aload1 = [&](uint32_t stage, int lo, int q) {
    const int i = lo + q / PL, p = q % PL;
    fa[p][i] = *reinterpret_cast<const bf16x8 *>(smem + stage * STAGE + aoff + p * PLANE + i * 16 * RB);
  };
  auto bload1 = [&](uint32_t stage, auto par, int q) {
    const int p = q / FN, j = q % FN;
    fb[decltype(par)::value][p][j] =
        *reinterpret_cast<const bf16x8 *>(smem + stage * STAGE + boff + p * PLANE + j * 16 * RB);
  };
  v4f acc[FM][FN];
  constexpr bool F64 = FLUSH > 0;
  v4d acc64[F64 ? FM : 1][F64 ? FN : 1];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      acc[i][j] = v4f{};
      if constexpr (F64) acc64[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    }
  // the products of the rows [lo, hi) of A; hook(n) runs after the n-th MFMA
  auto mfma = [&](auto par, auto lo, auto hi, auto fold, auto &&hook) {
    constexpr int L0 = decltype(lo)::value, NR = decltype(hi)::value - L0;
#pragma unroll
    for (int n = 0; n < NTERM * NR * FN; ++n) {
      const int t = n / (NR * FN), i = L0 + n / FN % NR, j = n % FN;
      if constexpr (decltype(fold)::value) {
        if (t == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc64[i][j][e] += double(acc[i][j][e]);
          acc[i][j] = v4f{};
        }
      }
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[TA[t]][i], fb[decltype(par)::value][TB[t]][j], acc[i][j],
                                                          0, 0, 0);
      hook(n);
    }
  };
  constexpr auto I0 = std::integral_constant<int, 0>{};
  constexpr auto I1 = std::integral_constant<int, 1>{};
  constexpr auto IH = std::integral_constant<int, HM>{};
  constexpr auto IF = std::integral_constant<int, FM>{};
  constexpr auto NO = std::false_type{};
  auto barrier = [&] {   // waits for this wave's LDS reads, not for its loads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  auto phase = [] { __builtin_amdgcn_sched_barrier(0); };
  const uint32_t last = ktiles - 1;
  uint32_t cur = 0;   // stage of tile kt
  constexpr int NM = NTERM * HM * FN;   // MFMAs of one phase
  auto body = [&](uint32_t kt, auto par, auto fold) {
    constexpr int P = decltype(par)::value;
    constexpr auto PN = std::integral_constant<int, P ^ 1>{};
    constexpr int NR = PL * (HM + FN);        // LDS reads of the second phase
    constexpr int DS = NM / PERT;             // MFMAs per load
    static_assert(DS >= 1 && NM > 4, "phase too short");
    auto ahead = [&] {   // bytes into a row; past the end: the last tile again, never read
      const uint32_t kn = kt + NST < last ? kt + NST : last;
      return uint64_t(kn) * RB;
    };
    mfma(par, I0, IH, fold, [&](int n) {
      bool any = n < PL * HM;
      if (n < PL * HM) aload1(cur, HM, n);
      if constexpr (!DMA) {
        if (n % DS == DS / 2 && n / DS < PERT) {
          put1(cur ^ 1, n / DS);
          fetch1(ahead(), n / DS);
          any = true;
        }
      }
      if (any) phase();
    });
    phase();
    // this wave's part of tile kt + 1 has landed; past the barrier all of it
    // has, and no wave reads the stage of tile kt any more
    const uint32_t nxt = cur + 1 == NST ? 0 : cur + 1;
    if constexpr (DMA) wait_vm<(NST - 2) * PERT>();
    barrier();
    phase();
    const uint64_t kb = ahead();
    const uint32_t base = lds0 + cur * STAGE;
    mfma(par, IH, IF, fold, [&](int n) {
      bool any = false;
#pragma unroll
      for (int q = n * NR / (NM - 4); q < (n + 1) * NR / (NM - 4) && q < NR; ++q) {
        if (q < PL * FN) bload1(nxt, PN, q);
        else aload1(nxt, 0, q - PL * FN);
        any = true;
      }
      if constexpr (DMA) {
        if (n % DS == DS / 2 && n / DS < PERT) {
          dma1(kb, base, n / DS);
          any = true;
        }
      }
      if (any) phase();
    });
    phase();
    cur = nxt;
  };
  if constexpr (DMA) {
#pragma unroll
    for (int s = 0; s < NST; ++s) dma(uint32_t(s) < last ? s : last, s);
    wait_vm<(NST - 1) * PERT>();
  } else {
#pragma unroll
    for (int q = 0; q < PERT; ++q) fetch1(0, q);
#pragma unroll
    for (int q = 0; q < PERT; ++q) put1(0, q);
#pragma unroll
    for (int q = 0; q < PERT; ++q) fetch1(last > 0 ? RB : 0, q);
  }
  barrier();
#pragma unroll
  for (int q = 0; q < PL * HM; ++q) aload1(0, 0, q);
#pragma unroll
  for (int q = 0; q < PL * FN; ++q) bload1(0, I0, q);
  constexpr auto FD = std::integral_constant<bool, F64>{};
  if constexpr (DMA) {
    for (uint32_t kt = 0;; kt += 4) {
      body(kt, I0, FD);
      if (kt == last) break;
      body(kt + 1, I1, NO);
      if (kt + 1 == last) break;
      body(kt + 2, I0, NO);
      if (kt + 2 == last) break;
      body(kt + 3, I1, NO);
      if (kt + 3 == last) break;
    }
  } else {   // four tiles without an exit, past which the compiler would move their loads and reads
    uint32_t kt = 0;
    for (; kt + 4 <= ktiles; kt += 4) {
      body(kt, I0, FD);
      body(kt + 1, I1, NO);
      body(kt + 2, I0, NO);
      body(kt + 3, I1, NO);
    }
    if (kt < ktiles) body(kt, I0, FD);
    if (kt + 1 < ktiles) body(kt + 1, I1, NO);
    if (kt + 2 < ktiles) body(kt + 2, I0, NO);
  }
  wait_vm<0>();
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float *dst = C + (m0 + wm * TM + i * 16 + 4 * g + e) * ldc + n0 + wn * TN + j * 16 + r16;
        if constexpr (F64) {
          const double v = acc64[i][j][e] + double(acc[i][j][e]);
          *dst = ACCUM ? float(double(*dst) + v) : float(v);
        } else {
          *dst = ACCUM ? *dst + acc[i][j][e] : acc[i][j][e];
        }
      }
}

template <int PREC, int BM, int BN, int WM, int WN, int MINW>
void launch_pipe(const void *A, const void *Bt, void *C, uint64_t M, uint64_t N, uint64_t K, uint64_t lda,
                 uint64_t ldb, uint64_t ldc, bool accum, hipStream_t st, uint32_t splits, uint64_t c_split_stride,
                 uint32_t nb, uint64_t batch_a, uint64_t batch_b, uint64_t batch_c) {
  using in_t = typename Prec<PREC>::in_t;
  using out_t = typename Prec<PREC>::out_t;
  constexpr size_t lds = 2 * size_t(BM + BN) * 128;
  constexpr int BK = 128 / Prec<PREC>::elem;
  static const bool attr = [] {   // dynamic LDS above 64 KB must be allowed per kernel
    TRG_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_pipe_kernel<PREC, BM, BN, WM, WN, MINW, true>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    TRG_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_pipe_kernel<PREC, BM, BN, WM, WN, MINW, false>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    return true;
  }();
  (void)attr;
  const uint32_t tm = uint32_t(M / BM), tn = uint32_t(N / BN), kt = uint32_t(K / BK / splits);
  const dim3 grid(tm * tn, splits, nb), block(64 * WM * WN);
  auto *a = static_cast<const in_t *>(A);
  auto *b = static_cast<const in_t *>(Bt);
  auto *c = static_cast<out_t *>(C);
  if (accum)
    hipLaunchKernelGGL((gemm_pipe_kernel<PREC, BM, BN, WM, WN, MINW, true>), grid, block, lds, st, a, b, c, tm, tn, kt,
                       lda, ldb, ldc, c_split_stride, batch_a, batch_b, batch_c, RowsRight{});
  else
    hipLaunchKernelGGL((gemm_pipe_kernel<PREC, BM, BN, WM, WN, MINW, false>), grid, block, lds, st, a, b, c, tm, tn,
                       kt, lda, ldb, ldc, c_split_stride, batch_a, batch_b, batch_c, RowsRight{});
  TRG_HIP_CHECK(hipGetLastError());
}

template <int BM, int BN, int MINW, bool PAIRS>
void launch_cols(const double *A, const double *B, double *C, uint64_t lda, uint32_t splits, uint32_t kt,
                 const ColsRight<PAIRS> &rt, hipStream_t st) {
  constexpr size_t lds = 2 * (size_t(BM) * 128 + 16 * size_t(BN + 4) * 8);
  auto *kernel = &gemm_pipe_kernel<0, BM, BN, 2, 2, MINW, false, ColsRight<PAIRS>>;
  static const bool attr = [kernel] {
    TRG_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    return true;
  }();
  (void)attr;
  const uint32_t tm = (rt.M + BM - 1) / BM, tn = (rt.N + BN - 1) / BN;
  hipLaunchKernelGGL(kernel, dim3(tm * tn, splits), dim3(256), lds, st, A, B, C, tm, tn, kt, lda, uint64_t(0),
                     uint64_t(rt.N), uint64_t(rt.M) * rt.N, uint64_t(0), uint64_t(0), uint64_t(0), rt);
  TRG_HIP_CHECK(hipGetLastError());
}

// ------------------------------------------------------ small FP64 products ---
// One 32 x 32 tile per workgroup of KSP_WAVES waves that share its K: wave w
// takes the K chunks (16 doubles) w, w + KSP_WAVES, ... straight from memory
// into MFMA fragments (no LDS, no barrier; KSP_DEPTH chunks in flight), and the
// waves' sums are added in a fixed order through LDS.  For products whose
// tiles do not fill the chip (2D joins: M = N = 256, K = 2752 is 16 tiles of
// 64 x 64), where the length of the K loop of one wave is what takes the time.
constexpr int KSP_WAVES = 8, KSP_DEPTH = 4, KSP_T = 32;

template <bool ACCUM>
__global__ void __launch_bounds__(64 * KSP_WAVES)
gemm_ksplit_kernel(const double *__restrict__ A, const double *__restrict__ Bt, double *__restrict__ C,
                   uint32_t tiles_n, uint32_t chunks, uint64_t lda, uint64_t ldb, uint64_t ldc, uint64_t c_split_stride,
                   uint64_t batch_a, uint64_t batch_b, uint64_t batch_c) {
  __shared__ double part[KSP_WAVES][KSP_T * KSP_T];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, r16 = lane & 15;
  const uint64_t m0 = uint64_t(blockIdx.x / tiles_n) * KSP_T, n0 = uint64_t(blockIdx.x % tiles_n) * KSP_T;
  const uint64_t koff = uint64_t(blockIdx.y) * chunks * 16 + 2 * g;
  const double *a0 = A + uint64_t(blockIdx.z) * batch_a + (m0 + r16) * lda + koff;
  const double *b0 = Bt + uint64_t(blockIdx.z) * batch_b + (n0 + r16) * ldb + koff;
  C += uint64_t(blockIdx.z) * batch_c + uint64_t(blockIdx.y) * c_split_stride;
  // lane group g holds k = 2 g, 2 g + 1 and 8 + 2 g, 9 + 2 g of a chunk
  d2 fa[KSP_DEPTH][2][2], fb[KSP_DEPTH][2][2];
  auto load = [&](uint32_t c, auto slot) {
    constexpr int s = decltype(slot)::value;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        fa[s][i][f] = *reinterpret_cast<const d2 *>(a0 + uint64_t(16 * i) * lda + uint64_t(c) * 16 + 8 * f);
        fb[s][i][f] = *reinterpret_cast<const d2 *>(b0 + uint64_t(16 * i) * ldb + uint64_t(c) * 16 + 8 * f);
      }
  };
  v4d acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  auto mul = [&](auto slot) {
    constexpr int s = decltype(slot)::value;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s][i][f][e], fb[s][j][f][e], acc[i][j], 0, 0, 0);
  };
  auto each_slot = [&](auto &&fn) {
    fn(std::integral_constant<int, 0>{});
    fn(std::integral_constant<int, 1>{});
    fn(std::integral_constant<int, 2>{});
    fn(std::integral_constant<int, 3>{});
  };
  static_assert(KSP_DEPTH == 4, "each_slot lists the slots");
  const uint32_t mine = chunks > uint32_t(wave) ? (chunks - wave + KSP_WAVES - 1) / KSP_WAVES : 0;   // chunks of this wave
  auto chunk = [&](uint32_t q) { return wave + q * KSP_WAVES; };
  each_slot([&](auto s) {
    if (uint32_t(decltype(s)::value) < mine) load(chunk(decltype(s)::value), s);
  });
  uint32_t q = 0;
  for (; q + 2 * KSP_DEPTH <= mine; q += KSP_DEPTH)
    each_slot([&](auto s) {
      mul(s);
      load(chunk(q + KSP_DEPTH + decltype(s)::value), s);
    });
  for (; q < mine; q += KSP_DEPTH)   // fewer than 2 KSP_DEPTH chunks left
    each_slot([&](auto s) {
      constexpr uint32_t u = decltype(s)::value;
      if (q + u < mine) mul(s);
      if (q + KSP_DEPTH + u < mine) load(chunk(q + KSP_DEPTH + u), s);
    });
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wave][(16 * i + g + 4 * e) * KSP_T + 16 * j + r16] = acc[i][j][e];
  __syncthreads();
  for (int o = threadIdx.x; o < KSP_T * KSP_T; o += 64 * KSP_WAVES) {
    const int r = o / KSP_T, c = o % KSP_T;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < KSP_WAVES; ++w) v += part[w][r * KSP_T + c];
    double *dst = C + (m0 + r) * ldc + n0 + c;
    *dst = ACCUM ? *dst + v : v;
  }
}

void launch_ksplit(const double *A, const double *Bt, double *C, uint64_t M, uint64_t N, uint64_t K, uint64_t lda,
                   uint64_t ldb, uint64_t ldc, bool accum, hipStream_t st, uint32_t splits, uint64_t c_split_stride,
                   uint32_t nb, uint64_t batch_a, uint64_t batch_b, uint64_t batch_c) {
  const uint32_t tn = uint32_t(N / KSP_T), chunks = uint32_t(K / 16 / splits);
  const dim3 grid(uint32_t(M / KSP_T) * tn, splits, nb), block(64 * KSP_WAVES);
  if (accum)
    hipLaunchKernelGGL((gemm_ksplit_kernel<true>), grid, block, 0, st, A, Bt, C, tn, chunks, lda, ldb, ldc,
                       c_split_stride, batch_a, batch_b, batch_c);
  else
    hipLaunchKernelGGL((gemm_ksplit_kernel<false>), grid, block, 0, st, A, Bt, C, tn, chunks, lda, ldb, ldc,
                       c_split_stride, batch_a, batch_b, batch_c);
  TRG_HIP_CHECK(hipGetLastError());
}

// What every launch checks: K in `splits` equal ranges of whole K tiles,
// 16-byte aligned rows, batch strides that keep the products apart.  False:
// nothing to multiply (M, N or K zero; K = 0 clears C unless accumulating).
template <int PREC>
bool check_gemm(uint64_t BM, uint64_t BN, uint64_t BK, void *C, uint64_t M, uint64_t N, uint64_t K, uint64_t lda,
                uint64_t ldb, uint64_t ldc, bool accum, hipStream_t st, uint32_t splits, uint32_t nb, uint64_t batch_a,
                uint64_t batch_b, uint64_t batch_c) {
  using P = Prec<PREC>;
  using out_t = typename P::out_t;
  TRG_REQUIRE(M % BM == 0 && N % BN == 0 && K % BK == 0, "gemm: M, N, K must be tile multiples");
  TRG_REQUIRE(lda >= K && ldb >= K && ldc >= N, "gemm: leading dimension too small");
  TRG_REQUIRE((lda * P::elem) % 16 == 0 && (ldb * P::elem) % 16 == 0, "gemm: rows must be 16-byte aligned");
  if (M == 0 || N == 0) return false;
  TRG_REQUIRE((M / BM) * (N / BN) < (1ull << 31) && K / BK < (1ull << 31), "gemm: problem too large for one launch");
  TRG_REQUIRE(nb >= 1 && nb <= 65535, "gemm: batch size out of range");
  TRG_REQUIRE(nb == 1 || (batch_a >= M * lda * P::planes && batch_b >= N * ldb * P::planes && batch_c >= M * ldc),
              "gemm: batch strides overlap the products");
  if (K == 0) {
    if (!accum)
      for (uint32_t b = 0; b < nb; ++b) fill_zero(static_cast<out_t *>(C) + b * batch_c, sizeof(out_t) * M * ldc, st);
    return false;
  }
  TRG_REQUIRE(splits >= 1 && K % (uint64_t(splits) * BK) == 0, "gemm: K not divisible by splits");
  return true;
}

template <int PL, int BM, int BN, int WM, int WN, int NST, int FLUSH, bool DMA = true>
void launch_split(const void *A, const void *Bt, void *C, uint64_t M, uint64_t N, uint64_t K, uint64_t lda,
                  uint64_t ldb, uint64_t ldc, bool accum, hipStream_t st, uint32_t nb, uint64_t batch_a,
                  uint64_t batch_b, uint64_t batch_c) {
  constexpr size_t lds = NST * size_t(BM + BN) * 64 * PL;
  static_assert(lds <= 160 * 1024, "LDS tile exceeds 160 KB");
  static const bool attr = [] {   // dynamic LDS above 64 KB must be allowed per kernel
    TRG_HIP_CHECK(hipFuncSetAttribute(
        reinterpret_cast<const void *>(&gemm_split_kernel<PL, BM, BN, WM, WN, NST, FLUSH, DMA, true>),
        hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    TRG_HIP_CHECK(hipFuncSetAttribute(
        reinterpret_cast<const void *>(&gemm_split_kernel<PL, BM, BN, WM, WN, NST, FLUSH, DMA, false>),
        hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    return true;
  }();
  (void)attr;
  const uint32_t tm = uint32_t(M / BM), tn = uint32_t(N / BN), kt = uint32_t(K / 32);
  const dim3 grid(tm * tn, 1, nb), block(64 * WM * WN);
  auto *a = static_cast<const uint16_t *>(A);
  auto *b = static_cast<const uint16_t *>(Bt);
  auto *c = static_cast<float *>(C);
  const uint64_t plA = M * lda, plB = N * ldb;
  if (accum)
    hipLaunchKernelGGL((gemm_split_kernel<PL, BM, BN, WM, WN, NST, FLUSH, DMA, true>), grid, block, lds, st, a, b, c, tm, tn,
                       kt, lda, ldb, ldc, plA, plB, batch_a, batch_b, batch_c);
  else
    hipLaunchKernelGGL((gemm_split_kernel<PL, BM, BN, WM, WN, NST, FLUSH, DMA, false>), grid, block, lds, st, a, b, c, tm,
                       tn, kt, lda, ldb, ldc, plA, plB, batch_a, batch_b, batch_c);
  TRG_HIP_CHECK(hipGetLastError());
}

}  // namespace

GemmTile gemm_tile(int prec) {
  switch (prec) {
    case 0: return {128, 128, 16};
    case 1: return {128, 128, 32};
    case 2: return {256, 256, 32};
    case 3: return {128, 128, 32};
  }
  throw Error(-1, "gemm: unknown precision");
}

namespace {

// FP64 products: the tile whose last round wastes least.  A launch takes about
// ceil(tiles / 256 CUs) times the time of one tile, tile area over the rate of
// the kernel on full rounds (measured on M = N = 8192, 3200 and 1024: 128 x 128
// 74 TFLOP/s, 64 x 128 70, 64 x 64 66, K split in the workgroup 50):
//   M = N = 10112 (K 25008)  128 x 128 72.3, 64 x 128 65.7, 64 x 64 64.1 TFLOP/s
//   M = N = 3200 (K 3136)    128 x 128 59.7, 64 x 128 69.9, 64 x 64 65.7
//   M = N = 1024 (K 1024)    128 x 128 17.4, 64 x 128 31.4, 64 x 64 49.8
//   M = N = 256 (K 2752)     64 x 64 3.6, K split 8.6
double f64_cost(uint64_t M, uint64_t N, double count, uint64_t bm, uint64_t bn, double rate) {
  if (M % bm || N % bn) return 1e300;
  return std::ceil(double(M / bm) * double(N / bn) * count / 256.0) * double(bm * bn) / rate;
}
constexpr double RATE_128 = 74.0, RATE_64_128 = 70.0, RATE_64 = 66.0, RATE_KSPLIT = 50.0;

void gemm_f64(const void *A, const void *Bt, void *C, uint64_t M, uint64_t N, uint64_t K, uint64_t lda, uint64_t ldb,
              uint64_t ldc, bool accum, hipStream_t st, uint32_t splits, uint64_t c_split_stride, uint32_t nb,
              uint64_t batch_a, uint64_t batch_b, uint64_t batch_c, bool ksplit) {
  if (ksplit) {
    launch_ksplit(static_cast<const double *>(A), static_cast<const double *>(Bt), static_cast<double *>(C), M, N, K,
                  lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a, batch_b, batch_c);
    return;
  }
  const double count = double(splits) * nb;
  const double c128 = f64_cost(M, N, count, 128, 128, RATE_128), c64 = f64_cost(M, N, count, 64, 128, RATE_64_128);
  const double c6464 = f64_cost(M, N, count, 64, 64, RATE_64);
  if (c128 <= c64 && c128 <= c6464)
    launch_pipe<0, 128, 128, 2, 2, 2>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a,
                                      batch_b, batch_c);
  else if (c64 <= c6464)
    launch_pipe<0, 64, 128, 2, 2, 3>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a,
                                     batch_b, batch_c);
  else
    launch_pipe<0, 64, 64, 2, 2, 4>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a,
                                    batch_b, batch_c);
}

// Split-BF16 products: whether tiles of `small` squared finish before tiles of
// `big` squared, whose last round may leave most of the 256 CUs idle; `rate`
// is the speed of the small-tile kernel over the big-tile one on full rounds.
// BF16x6, 64 x 64 against 128 x 128 tiles, TFLOP/s: 512^2 x 1024 44 and 18,
// 1024^2 x 1024 115 and 67, 1280^2 x 1024 115 and 104, 1664^2 x 1664 132 and 170,
// 2176^2 x 2048 130 and 146, 7808^2 x 7776 116 and 192, 10112^2 x 25056 110 and 188.
bool split_small(uint64_t M, uint64_t N, uint32_t nb, uint64_t big, uint64_t small, double rate) {
  auto cost = [&](uint64_t b) { return std::ceil(double(M / b) * double(N / b) * nb / 256.0) * double(b * b); };
  return cost(small) < rate * cost(big);
}

// Whether every row of both split-BF16 operands starts on 16 bytes (the rows
// of a plane and the planes are multiples of that apart: check_gemm).  Others
// go through registers, at 60 to 75 % of the rate.
bool split_direct(const void *A, const void *Bt, uint32_t nb, uint64_t batch_a, uint64_t batch_b) {
  const bool bases = (reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(Bt)) % 16 == 0;
  return bases && (nb == 1 || (batch_a * 2 % 16 == 0 && batch_b * 2 % 16 == 0));
}

}  // namespace

bool gemm_f64_ksplit(uint64_t M, uint64_t N, uint64_t K) {
  if (M % KSP_T || N % KSP_T || K < 16 * 2 * KSP_WAVES) return false;   // a few chunks per wave
  const double tiled = std::min(std::min(f64_cost(M, N, 1, 128, 128, RATE_128), f64_cost(M, N, 1, 64, 128, RATE_64_128)),
                                f64_cost(M, N, 1, 64, 64, RATE_64));
  return f64_cost(M, N, 1, KSP_T, KSP_T, RATE_KSPLIT) < tiled;
}

void gemm_nt(int prec, const void *A, const void *Bt, void *C, uint64_t M, uint64_t N, uint64_t K,
             uint64_t lda, uint64_t ldb, uint64_t ldc, bool accum, hipStream_t st, uint32_t nb, uint64_t batch_a,
             uint64_t batch_b, uint64_t batch_c, int ksplit) {
  switch (prec) {
    case 0:
      if (check_gemm<0>(128, 128, 16, C, M, N, K, lda, ldb, ldc, accum, st, 1, nb, batch_a, batch_b, batch_c))
        gemm_f64(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, 1, 0, nb, batch_a, batch_b, batch_c,
                 ksplit < 0 ? gemm_f64_ksplit(M, N, K) : ksplit != 0);
      return;
    case 1:
      if (!check_gemm<1>(128, 128, 32, C, M, N, K, lda, ldb, ldc, accum, st, 1, nb, batch_a, batch_b, batch_c)) return;
      // 64 x 64 tiles while 64 x 128 ones leave CUs idle (M = N = K = 1024:
      // 97 against 54 TFLOP/s; M = N = 7808: 130 against 132)
      if ((M / 64) * (N / 128) * nb <= 512)
        launch_pipe<1, 64, 64, 2, 2, 2>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, 1, 0, nb, batch_a, batch_b, batch_c);
      else
        launch_pipe<1, 64, 128, 2, 2, 2>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, 1, 0, nb, batch_a, batch_b, batch_c);
      return;
    case 2:
      if (!check_gemm<2>(256, 256, 32, C, M, N, K, lda, ldb, ldc, accum, st, 1, nb, batch_a, batch_b, batch_c)) return;
      if (!split_direct(A, Bt, nb, batch_a, batch_b)) {
        // 128 x 256 tiles once they fill three quarters of the CUs, against 128 x 128 ones:
        // 2048^2 x 4096 211 and 249 TFLOP/s, 3072 x 2048 x 4096 290 and 230, 4096^2 x 6400 351 and 291
        if ((M / 128) * (N / 256) * nb >= 192)
          launch_split<2, 128, 256, 2, 4, 2, 0, false>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a, batch_b,
                                                       batch_c);
        else
          launch_split<2, 128, 128, 2, 2, 2, 0, false>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a, batch_b,
                                                       batch_c);
        return;
      }
      // four waves of 64 x 64, two workgroups per CU, while the 256 x 256 tiles leave CUs idle in
      // their last round: 2048^2 x 8192 338 against 186 TFLOP/s, 10240^2 x 25056 290 against 407
      if (split_small(M, N, nb, 256, 128, 290.0 / 407.0))
        launch_split<2, 128, 128, 2, 2, 2, 0>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a, batch_b, batch_c);
      else
        launch_split<2, 256, 256, 2, 4, 2, 0>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a, batch_b, batch_c);
      return;
    case 3:
      if (!check_gemm<3>(128, 128, 32, C, M, N, K, lda, ldb, ldc, accum, st, 1, nb, batch_a, batch_b, batch_c)) return;
      if (!split_direct(A, Bt, nb, batch_a, batch_b))
        launch_split<3, 128, 128, 2, 4, 2, BF6_FLUSH, false>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a,
                                                           batch_b, batch_c);
      else if (split_small(M, N, nb, 128, 64, 0.6))
        launch_split<3, 64, 64, 2, 2, 3, BF6_FLUSH>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a, batch_b,
                                                    batch_c);
      else
        launch_split<3, 128, 128, 2, 4, 3, BF6_FLUSH>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a, batch_b,
                                                      batch_c);
      return;
  }
  throw Error(-1, "gemm: unknown precision");
}

// Split-K FP64 products of the Gram reductions: split s covers K range
// [s*kper, (s+1)*kper) and writes its own M x N slab of Cpart.  M and N are
// multiples of 64; K must equal splits * kper (zero-padded).
void gemm_nt_splitk_f64(const double *A, const double *Bt, double *Cpart, uint64_t M, uint64_t N,
                        uint64_t K, uint64_t lda, uint64_t ldb, uint32_t splits, uint64_t kper,
                        hipStream_t st) {
  TRG_REQUIRE(K == uint64_t(splits) * kper, "splitk: K != splits * kper");
  if (check_gemm<0>(64, 64, 16, Cpart, M, N, K, lda, ldb, N, false, st, splits, 1, 0, 0, 0))
    gemm_f64(A, Bt, Cpart, M, N, K, lda, ldb, N, false, st, splits, M * N, 1, 0, 0, 0, false);
}

// Tile and number of K ranges of a product with a column-contiguous right
// operand, by the time of its rounds on 256 CUs (tile area times the length of
// a range over the rate of the tile, as for the other FP64 products) and, with
// several ranges, the traffic of the partial sums (4 TB/s) and their launch.
ColsPlan gemm_cols_plan(uint64_t M, uint64_t N, uint64_t K) {
  struct Tile {
    uint64_t bm, bn;
    double rate;
  };
  constexpr Tile tiles[3] = {{128, 128, RATE_128}, {64, 128, RATE_64_128}, {64, 64, RATE_64}};
  const uint64_t kt = (K + 15) / 16;
  ColsPlan best{};
  double tbest = 1e300;
  for (int i = 0; i < 3; ++i) {
    const Tile &t = tiles[i];
    const uint64_t n = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    for (uint64_t want = 1; want <= 32 && want <= kt; ++want) {
      const uint64_t per = (kt + want - 1) / want, splits = (kt + per - 1) / per;
      double time = std::ceil(double(n) * double(splits) / 256.0) * double(t.bm * t.bn * 2 * 16) * double(per) * 256.0 /
                    (t.rate * 1e12);
      if (splits > 1) time += 5e-6 + double(splits + 1) * double(M) * double(N) * 8.0 / 4e12;
      if (time < tbest) {
        tbest = time;
        best = ColsPlan{i, uint32_t(splits), uint32_t(per)};
      }
    }
  }
  return best;
}

// C[m][n] = sum_k A[m][k] B(k, n): A K-contiguous with pitch lda, its rows
// zero-padded to a multiple of 128 and its columns to one of 16; B as described
// at ColsRight; C (M x N, unpadded) or, with several K ranges, `part` receives
// one M x N slab per range, summed into C in order.
void gemm_cols_f64(const ColsPlan &plan, const double *A, uint64_t lda, const double *B, const ColsShape &s, double *C,
                   double *part, hipStream_t st) {
  constexpr uint64_t lim = uint64_t(1) << 31;
  TRG_REQUIRE(s.M >= 1 && s.N >= 1 && s.K >= 1 && s.M < lim && s.N < lim && s.K < lim && s.k1 >= 1 && s.n1 >= 1 &&
                  s.k1 <= s.K && s.n1 <= s.N,
              "gemm_cols: bad shape");
  TRG_REQUIRE(lda % 2 == 0 && lda >= (s.K + 15) / 16 * 16, "gemm_cols: bad left operand");
  TRG_REQUIRE(plan.splits >= 1 && uint64_t(plan.splits - 1) * plan.ktiles < (s.K + 15) / 16 &&
                  uint64_t(plan.splits) * plan.ktiles >= (s.K + 15) / 16 && (plan.splits == 1 || part),
              "gemm_cols: bad plan");
  TRG_REQUIRE(((s.M + 63) / 64) * ((s.N + 63) / 64) < lim, "gemm_cols: too many tiles");
  const bool pairs = s.N % 2 == 0 && s.n1 % 2 == 0 && s.sk1 % 2 == 0 && s.sk2 % 2 == 0 && s.sn2 % 2 == 0 &&
                     reinterpret_cast<uintptr_t>(B) % 16 == 0;
  double *out = plan.splits > 1 ? part : C;
  auto launch = [&](auto rt) {
    constexpr bool P = decltype(rt)::pairs;
    rt.M = uint32_t(s.M);
    rt.N = uint32_t(s.N);
    rt.K = uint32_t(s.K);
    rt.k1 = uint32_t(s.k1);
    rt.n1 = uint32_t(s.n1);
    rt.sk1 = s.sk1;
    rt.sk2 = s.sk2;
    rt.sn2 = s.sn2;
    if (plan.tile == 0) launch_cols<128, 128, 2, P>(A, B, out, lda, plan.splits, plan.ktiles, rt, st);
    else if (plan.tile == 1) launch_cols<64, 128, 3, P>(A, B, out, lda, plan.splits, plan.ktiles, rt, st);
    else launch_cols<64, 64, 4, P>(A, B, out, lda, plan.splits, plan.ktiles, rt, st);
  };
  if (pairs) launch(ColsRight<true>{});
  else launch(ColsRight<false>{});
  if (plan.splits > 1)
    reduce_splits(part, int(plan.splits), int64_t(s.M), int64_t(s.N), int64_t(s.N), int64_t(s.M * s.N), C, int64_t(s.N),
                  st);
}

}  // namespace trg
