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
//   BF16X3 v_mfma_f32_16x16x32_bf16 256 x 256 tile, eight 128 x 64 waves,
//          RB 64 (32 bf16 per plane, 1 k-step, three products hi*hi +
//          hi*lo + lo*hi into one FP32 accumulator), two swizzled stages
//   BF16X6 v_mfma_f32_16x16x32_bf16 128 x 128 tile, eight 64 x 32 waves,
//          RB 64, three planes (fl32(a) = hi + mid + lo exactly), six
//          products hi*hi + hi*mid + mid*hi + mid*mid + hi*lo + lo*hi; the
//          MFMA sums BF6_FLUSH K tiles in FP32, the groups are summed in
//          FP64 (FP32-accurate operands and FP64-grade accumulation), two
//          swizzled stages
//
// Two LDS stages: the next tile's global loads are in flight while the
// current tile feeds the MFMAs (one barrier per tile).
//
// Workgroup ids are remapped so that each XCD (ids are dealt round-robin to
// the 8 XCDs) works on one contiguous range of tiles, walked in groups of
// GROUP_M tile-rows: neighbouring tiles on one XCD share A and Bt rows in
// that XCD's L2.
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

constexpr int NUM_XCD = 8;
// FP32 join: K tiles (32 floats each) summed by the MFMA in FP32 before the
// partial sum is added to the FP64 accumulator
constexpr uint32_t F32_FLUSH = 4;
#ifndef TRG_GROUP_M
#define TRG_GROUP_M 8
#endif
constexpr int GROUP_M = TRG_GROUP_M;

// BF16X6 join: K tiles (32 elements each) per FP32 group
#ifndef TRG_BF6_FLUSH
#define TRG_BF6_FLUSH 4
#endif
// BF16X6 join: global -> LDS prefetch distance in K tiles (1 or 2)
#ifndef TRG_BF6_PF
#define TRG_BF6_PF 2
#endif
constexpr uint32_t BF6_FLUSH = TRG_BF6_FLUSH;

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

// LDS layout of one operand tile: rows of RB bytes of K.  Padded (SWZ 0):
// row stride RB + 16.  Swizzled (SWZ 1): row stride RB, and the 16-byte
// chunk c of row r is stored at chunk c ^ ((r / (256 / RB)) % (RB / 16)).
// Either way the 16 rows that one lane group reads fall on 16 disjoint
// 4-bank groups of the 64-bank LDS; with the swizzle, 16 consecutive lanes
// also store 256 contiguous bytes (no padding, no store conflicts).
template <int RB, int SWZ>
__device__ inline int lds_off(int row, int chunk) {
  if constexpr (SWZ == 0) {
    return row * (RB + 16) + (chunk << 4);
  } else {
    constexpr int CPR = RB / 16, RPL = 256 / RB;
    return row * RB + ((chunk ^ ((row / RPL) % CPR)) << 4);
  }
}
template <int RB, int SWZ>
constexpr int lds_stride() { return SWZ ? RB : RB + 16; }

// BM x BN tile per workgroup, WM x WN waves of 64 lanes, K in tiles of RB
// bytes per row.
template <int PREC, int BM, int BN, int WM, int WN, int RB, int SWZ, int PF, bool ACCUM>
__global__ void __launch_bounds__(64 * WM * WN)
gemm_nt_kernel(const typename Prec<PREC>::in_t *__restrict__ A,
               const typename Prec<PREC>::in_t *__restrict__ Bt,
               typename Prec<PREC>::out_t *__restrict__ C, uint32_t tiles_m, uint32_t tiles_n,
               uint32_t ktiles, uint64_t lda, uint64_t ldb, uint64_t ldc, uint64_t planeA,
               uint64_t planeB, uint64_t batch_a, uint64_t batch_b, uint64_t batch_c) {
  using P = Prec<PREC>;
  using in_t = typename P::in_t;
  using acc_t = typename P::acc_t;
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;      // wave tile
  constexpr int FM = TM / 16, FN = TN / 16;      // 16x16 MFMA blocks per wave
  constexpr int PL = P::planes;
  constexpr int CPR = RB / 16;                   // 16-byte chunks per row
  constexpr int CH_A = BM * CPR;                 // chunks per A tile plane
  constexpr int CH_B = BN * CPR;
  static_assert(CH_A % NT == 0 && CH_B % NT == 0, "tile/threads mismatch");
  static_assert(RB == 64 || RB == 128, "RB must be 64 or 128");
  constexpr int LA = CH_A / NT, LB = CH_B / NT;  // chunks per thread
  constexpr int STR = lds_stride<RB, SWZ>();
  constexpr int STAGE = (BM + BN) * STR * PL;
  constexpr int NF = RB / 64;                    // 16-byte fragments per lane per block row

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int g = lane >> 4, r16 = lane & 15;

  uint32_t tm, tn;
  tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const uint64_t m0 = uint64_t(tm) * BM, n0 = uint64_t(tn) * BN;

  // batch: blockIdx.z selects a product of the strided batch (elements)
  A += uint64_t(blockIdx.z) * batch_a;
  Bt += uint64_t(blockIdx.z) * batch_b;
  C += uint64_t(blockIdx.z) * batch_c;
  const unsigned char *gA = reinterpret_cast<const unsigned char *>(A + m0 * lda);
  const unsigned char *gB = reinterpret_cast<const unsigned char *>(Bt + n0 * ldb);
  const uint64_t ldaB = lda * P::elem, ldbB = ldb * P::elem;
  const uint64_t plA = planeA * P::elem, plB = planeB * P::elem;

  // PF register sets for the global -> LDS staging: with PF = 2 the loads
  // of tile t are issued two compute phases before tile t is stored to LDS
  static_assert(PF == 1 || PF == 2, "prefetch distance 1 or 2");
  u32x4 ra[PF][PL][LA], rb[PF][PL][LB];

  auto gload = [&](uint32_t kt, int set) {
    const uint64_t kb = uint64_t(kt) * RB;
#pragma unroll
    for (int p = 0; p < PL; ++p) {
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int c = tid + i * NT, row = c / CPR, col = c % CPR;
        ra[set][p][i] = *reinterpret_cast<const u32x4 *>(gA + p * plA + row * ldaB + kb + col * 16);
      }
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int c = tid + i * NT, row = c / CPR, col = c % CPR;
        rb[set][p][i] = *reinterpret_cast<const u32x4 *>(gB + p * plB + row * ldbB + kb + col * 16);
      }
    }
  };
  auto sstore = [&](int stage, int set) {
    unsigned char *base = smem + stage * STAGE;
#pragma unroll
    for (int p = 0; p < PL; ++p) {
      unsigned char *sA = base + p * (BM + BN) * STR;
      unsigned char *sB = sA + BM * STR;
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int c = tid + i * NT, row = c / CPR, col = c % CPR;
        *reinterpret_cast<u32x4 *>(sA + lds_off<RB, SWZ>(row, col)) = ra[set][p][i];
      }
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int c = tid + i * NT, row = c / CPR, col = c % CPR;
        *reinterpret_cast<u32x4 *>(sB + lds_off<RB, SWZ>(row, col)) = rb[set][p][i];
      }
    }
  };

  acc_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = acc_t{};
  // BF16X6: the MFMA accumulates one group of K tiles in FP32, the groups are
  // summed in FP64, so the rounding of the sum no longer grows with the full
  // length of K
  constexpr bool F64SUM = PREC == 3;
  constexpr uint32_t FLUSH = BF6_FLUSH;
  v4d acc64[F64SUM ? FM : 1][F64SUM ? FN : 1];
  if constexpr (F64SUM) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc64[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  }

  // MFMAs of the tile in LDS stage `cur`, then the FP64 fold of a finished
  // group (K tile kt is the last of its group, or the last one)
  auto compute = [&](int cur, uint32_t kt) {
    const unsigned char *base = smem + cur * STAGE;
    // fragments: lane group g owns chunks [g NF, g NF + NF) of every row
    using frag_t = typename P::frag_t;
    frag_t fa[PL][FM][NF], fb[PL][FN][NF];
#pragma unroll
    for (int p = 0; p < PL; ++p) {
      const unsigned char *sA = base + p * (BM + BN) * STR;
      const unsigned char *sB = sA + BM * STR;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int f = 0; f < NF; ++f)
          fa[p][i][f] = *reinterpret_cast<const frag_t *>(sA + lds_off<RB, SWZ>(wm * TM + i * 16 + r16, g * NF + f));
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int f = 0; f < NF; ++f)
          fb[p][j][f] = *reinterpret_cast<const frag_t *>(sB + lds_off<RB, SWZ>(wn * TN + j * 16 + r16, g * NF + f));
    }

    if constexpr (PREC == 3) {
      static_assert(NF == 1, "BF16X6 uses one 32-element k-step per K tile");
      // the six products of each block, the small ones first; each term
      // sweeps all accumulators so consecutive MFMAs are independent
      constexpr int TA[6] = {2, 0, 1, 1, 0, 0}, TB[6] = {0, 2, 1, 0, 1, 0};  // lo*hi, hi*lo, mid*mid, mid*hi, hi*mid, hi*hi
#pragma unroll
      for (int term = 0; term < 6; ++term)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[TA[term]][i][0], fb[TB[term]][j][0], acc[i][j], 0, 0, 0);
    } else {
#pragma unroll
      // the three products of a block are spread over all accumulators so
      // that consecutive MFMAs never depend on each other
      for (int s = 0; s < NF; ++s)
#pragma unroll
        for (int term = 0; term < 3; ++term)
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
              const int pa = term == 0 ? 1 : 0, pb = term == 1 ? 1 : 0;  // lo*hi, hi*lo, hi*hi
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[pa][i][s], fb[pb][j][s], acc[i][j], 0, 0, 0);
            }
    }

    if constexpr (F64SUM) {
      if ((kt + 1) % FLUSH == 0 || kt + 1 == ktiles) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc64[i][j][e] += double(acc[i][j][e]);
            acc[i][j] = acc_t{};
          }
      }
    }
  };

  if constexpr (PF == 2) {
    // tile t: registers set t % 2, LDS stage t % 2.  Iteration t issues the
    // loads of tile t + 2 into the set that tile t has left, computes stage
    // t % 2, then stores tile t + 1 (loaded during iteration t - 1) into the
    // stage that iteration t - 1 computed; one barrier per tile.  The main
    // loop has no conditional loads or stores, so the wait before a store
    // leaves the six loads issued after it in flight; the last one to three
    // tiles run in a tail with the bounds checks.
    gload(0, 0);
    sstore(0, 0);
    if (ktiles > 1) gload(1, 1);
    __syncthreads();
    auto body = [&](uint32_t kt, auto half) {
      constexpr int h = decltype(half)::value;
      gload(kt + 2, h);
      // keep the loads ahead of the MFMAs: the compiler would otherwise sink
      // them towards their use and shorten the prefetch distance to one tile
      // (the empty asm with a memory clobber stops sinking in the IR, the
      // scheduling barrier reordering in the machine scheduler)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      compute(h, kt);
      sstore(h ^ 1, h ^ 1);
      __syncthreads();
    };
    auto tail = [&](uint32_t kt, auto half) {
      constexpr int h = decltype(half)::value;
      if (kt + 2 < ktiles) gload(kt + 2, h);
      compute(h, kt);
      if (kt + 1 < ktiles) sstore(h ^ 1, h ^ 1);
      __syncthreads();
    };
    uint32_t kt = 0;
    for (; kt + 3 < ktiles; kt += 2) {
      body(kt, std::integral_constant<int, 0>{});
      body(kt + 1, std::integral_constant<int, 1>{});
    }
    // kt is even here and 1 to 3 tiles remain
    tail(kt, std::integral_constant<int, 0>{});
    if (kt + 1 < ktiles) tail(kt + 1, std::integral_constant<int, 1>{});
    if (kt + 2 < ktiles) tail(kt + 2, std::integral_constant<int, 0>{});
  } else {
    gload(0, 0);
    sstore(0, 0);
    __syncthreads();
    for (uint32_t kt = 0; kt < ktiles; ++kt) {
      const int cur = kt & 1;
      if (kt + 1 < ktiles) gload(kt + 1, 0);
      compute(cur, kt);
      if (kt + 1 < ktiles) sstore(cur ^ 1, 0);
      __syncthreads();
    }
  }

  // epilogue: register e of lane (g, r16) holds column r16, row 4g + e of each
  // 16x16 block
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 4 * g + e;
        const uint64_t m = m0 + wm * TM + i * 16 + row;
        const uint64_t n = n0 + wn * TN + j * 16 + r16;
        auto *dst = C + m * ldc + n;
        if constexpr (F64SUM) {
          if constexpr (ACCUM)
            *dst = float(double(*dst) + acc64[i][j][e]);
          else
            *dst = float(acc64[i][j][e]);
        } else {
          if constexpr (ACCUM)
            *dst += acc[i][j][e];
          else
            *dst = acc[i][j][e];
        }
      }
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
// barrier is covered by another's MFMAs.
//
// Measured (M = N = 10112, K = 25008 / 25056): FP64 58.3 -> 72.3 TFLOP/s (92 %
// of 78.6; MFMA pipes busy 77 -> 96 % at 8192^2), FP32 96 -> 138 TFLOP/s
// (88 % of 157; busy 70 -> 91 %), against a kernel that read all fragments of a
// tile from LDS right before its MFMAs with one wave per SIMD (FP64) or two in
// step (FP32).  Of the FP32 gain, 129 -> 138 comes from adding a finished
// group to the FP64 sums block by block between the next tile's first MFMAs.
template <int PREC, int BM, int BN, int WM, int WN, int MINW, bool ACCUM>
__global__ void __launch_bounds__(64 * WM * WN, MINW)
gemm_pipe_kernel(const typename Prec<PREC>::in_t *__restrict__ A, const typename Prec<PREC>::in_t *__restrict__ Bt,
                 typename Prec<PREC>::out_t *__restrict__ C, uint32_t tiles_m, uint32_t tiles_n, uint32_t ktiles,
                 uint64_t lda, uint64_t ldb, uint64_t ldc, uint64_t c_split_stride, uint64_t batch_a,
                 uint64_t batch_b, uint64_t batch_c) {
  using P = Prec<PREC>;
  using acc_t = typename P::acc_t;
  using frag_t = typename P::frag_t;
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 16, FN = TN / 16;
  constexpr int RB = 128, CPR = 8, BK = RB / P::elem;
  constexpr int LA = BM * CPR / NT, LB = BN * CPR / NT;
  static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads mismatch");
  constexpr int STAGE = (BM + BN) * RB;
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

  u32x4 ra[LA], rb[LB];
  auto gload = [&](uint32_t kt) {
    const uint64_t kb = uint64_t(kt) * RB;
#pragma unroll
    for (int i = 0; i < LA; ++i) ra[i] = *reinterpret_cast<const u32x4 *>(gA + i * stepA + kb);
#pragma unroll
    for (int i = 0; i < LB; ++i) rb[i] = *reinterpret_cast<const u32x4 *>(gB + i * stepB + kb);
  };
  // rows of one thread differ by NT / 8, a multiple of 16: one swizzle for all
  static_assert((NT / CPR) % 16 == 0, "swizzle period");
  unsigned char *const sbase = smem + row0 * RB + ((col0 ^ pipe_swz(row0)) << 4);
  auto sstore = [&](int stage) {
#pragma unroll
    for (int i = 0; i < LA; ++i) *reinterpret_cast<u32x4 *>(sbase + stage * STAGE + i * (NT / CPR) * RB) = ra[i];
#pragma unroll
    for (int i = 0; i < LB; ++i)
      *reinterpret_cast<u32x4 *>(sbase + stage * STAGE + BM * RB + i * (NT / CPR) * RB) = rb[i];
  };
  // half f of a lane's K share of a row: chunk 2 g + f
  const int swz = pipe_swz(r16);
  const int fro[2] = {((2 * g) ^ swz) << 4, ((2 * g + 1) ^ swz) << 4};
  const int abase = (wm * TM + r16) * RB, bbase = BM * RB + (wn * TN + r16) * RB;
  frag_t fa[2][FM], fb[2][FN];
  auto fload = [&](int stage, auto half) {
    constexpr int f = decltype(half)::value;
    const unsigned char *s = smem + stage * STAGE + fro[f];
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[f][i] = *reinterpret_cast<const frag_t *>(s + abase + i * 16 * RB);
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[f][j] = *reinterpret_cast<const frag_t *>(s + bbase + j * 16 * RB);
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
  if (ktiles > 1) gload(1);
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
    while (kt + 2 < ktiles) body(kt++, NO, YES, YES);
    if (kt + 1 < ktiles) body(kt++, NO, YES, NO);
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
        auto *dst = C + (m0 + wm * TM + i * 16 + row) * ldc + n0 + wn * TN + j * 16 + r16;
        if constexpr (F64SUM)
          *dst = ACCUM ? float(double(*dst) + acc64[i][j][e]) : float(acc64[i][j][e]);
        else
          *dst = ACCUM ? *dst + acc[i][j][e] : acc[i][j][e];
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
                       lda, ldb, ldc, c_split_stride, batch_a, batch_b, batch_c);
  else
    hipLaunchKernelGGL((gemm_pipe_kernel<PREC, BM, BN, WM, WN, MINW, false>), grid, block, lds, st, a, b, c, tm, tn,
                       kt, lda, ldb, ldc, c_split_stride, batch_a, batch_b, batch_c);
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

template <int PREC, int BM, int BN, int WM, int WN, int RB, int SWZ, int PF>
void launch_gemm(const void *A, const void *Bt, void *C, uint64_t M, uint64_t N, uint64_t K,
                 uint64_t lda, uint64_t ldb, uint64_t ldc, bool accum, hipStream_t st, uint32_t nb, uint64_t batch_a,
                 uint64_t batch_b, uint64_t batch_c) {
  using P = Prec<PREC>;
  constexpr int BK = RB / P::elem;
  if (!check_gemm<PREC>(BM, BN, BK, C, M, N, K, lda, ldb, ldc, accum, st, 1, nb, batch_a, batch_b, batch_c)) return;
  constexpr size_t lds = 2 * size_t(BM + BN) * lds_stride<RB, SWZ>() * P::planes;
  static_assert(lds <= 160 * 1024, "LDS tile exceeds 160 KB");
  using in_t = typename P::in_t;
  using out_t = typename P::out_t;
  auto *a = static_cast<const in_t *>(A);
  auto *b = static_cast<const in_t *>(Bt);
  auto *c = static_cast<out_t *>(C);
  const uint64_t plA = M * lda, plB = N * ldb;
  const uint32_t tm = uint32_t(M / BM), tn = uint32_t(N / BN), kt = uint32_t(K / BK);
  dim3 grid(tm * tn, 1, nb), block(64 * WM * WN);
  // dynamic LDS above 64 KB must be allowed per kernel (once per instantiation)
  static bool attr_set = false;
  if (!attr_set) {
    TRG_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_nt_kernel<PREC, BM, BN, WM, WN, RB, SWZ, PF, true>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    TRG_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_nt_kernel<PREC, BM, BN, WM, WN, RB, SWZ, PF, false>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    attr_set = true;
  }
  if (accum)
    hipLaunchKernelGGL((gemm_nt_kernel<PREC, BM, BN, WM, WN, RB, SWZ, PF, true>), grid, block, lds, st, a, b, c, tm, tn,
                       kt, lda, ldb, ldc, plA, plB, batch_a, batch_b, batch_c);
  else
    hipLaunchKernelGGL((gemm_nt_kernel<PREC, BM, BN, WM, WN, RB, SWZ, PF, false>), grid, block, lds, st, a, b, c, tm,
                       tn, kt, lda, ldb, ldc, plA, plB, batch_a, batch_b, batch_c);
  TRG_HIP_CHECK(hipGetLastError());
}

}  // namespace

// BF16x3 join: 256 x 256 workgroup tile, eight waves of 128 x 64 (two per
// SIMD), 64-byte K rows (32 bf16 per plane), two swizzled LDS stages of
// 64 KB.  Measured against 128 x 128 tiles of four 64 x 64 waves with
// 128-byte rows: 1.6x the MFMA issue rate, 2.5x less L2 -> fabric traffic.
struct BF {
  static constexpr int BM = 256, BN = 256, WM = 2, WN = 4, RB = 64, SWZ = 1;
};
// BF16x6 join: 128 x 128 workgroup tile, eight waves of 64 x 32 (two per
// SIMD: 32 FP32 accumulators, 64 FP64 group sums, 18 operand fragments of
// 16 bytes per lane), 64-byte K rows of three planes, swizzled LDS stages of
// 48 KB.  Six products per three planes read from LDS: per MFMA it reads a
// third less LDS than the BF16x3 join's two-plane, three-product blocks.
struct BF6 {
  static constexpr int BM = 128, BN = 128, WM = 2, WN = 4, RB = 64, SWZ = 1, PF = TRG_BF6_PF;
};

GemmTile gemm_tile(int prec) {
  switch (prec) {
    case 0: return {128, 128, 16};
    case 1: return {128, 128, 32};
    case 2: return {BF::BM, BF::BN, BF::RB / 2};
    case 3: return {BF6::BM, BF6::BN, BF6::RB / 2};
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
// The K split needs a K of a few chunks per wave.
void gemm_f64(const void *A, const void *Bt, void *C, uint64_t M, uint64_t N, uint64_t K, uint64_t lda, uint64_t ldb,
              uint64_t ldc, bool accum, hipStream_t st, uint32_t splits, uint64_t c_split_stride, uint32_t nb,
              uint64_t batch_a, uint64_t batch_b, uint64_t batch_c) {
  auto cost = [&](uint64_t bm, uint64_t bn, double rate) {
    if (M % bm || N % bn) return 1e300;
    const double tiles = double(M / bm) * double(N / bn) * splits * nb;
    return std::ceil(tiles / 256.0) * double(bm * bn) / rate;
  };
  const double c128 = cost(128, 128, 74.0), c64 = cost(64, 128, 70.0), c6464 = cost(64, 64, 66.0);
  const double cks = K / splits >= 16 * 2 * KSP_WAVES ? cost(KSP_T, KSP_T, 50.0) : 1e300;
  const double best = std::min(std::min(c128, c64), std::min(c6464, cks));
  if (best == c128)
    launch_pipe<0, 128, 128, 2, 2, 2>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a,
                                      batch_b, batch_c);
  else if (best == c64)
    launch_pipe<0, 64, 128, 2, 2, 3>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a,
                                     batch_b, batch_c);
  else if (best == c6464)
    launch_pipe<0, 64, 64, 2, 2, 4>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a,
                                    batch_b, batch_c);
  else
    launch_ksplit(static_cast<const double *>(A), static_cast<const double *>(Bt), static_cast<double *>(C), M, N, K,
                  lda, ldb, ldc, accum, st, splits, c_split_stride, nb, batch_a, batch_b, batch_c);
}

}  // namespace

void gemm_nt(int prec, const void *A, const void *Bt, void *C, uint64_t M, uint64_t N, uint64_t K,
             uint64_t lda, uint64_t ldb, uint64_t ldc, bool accum, hipStream_t st, uint32_t nb, uint64_t batch_a,
             uint64_t batch_b, uint64_t batch_c) {
  switch (prec) {
    case 0:
      if (check_gemm<0>(128, 128, 16, C, M, N, K, lda, ldb, ldc, accum, st, 1, nb, batch_a, batch_b, batch_c))
        gemm_f64(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, 1, 0, nb, batch_a, batch_b, batch_c);
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
      launch_gemm<2, BF::BM, BF::BN, BF::WM, BF::WN, BF::RB, BF::SWZ, 1>(A, Bt, C, M, N, K, lda, ldb, ldc, accum, st,
                                                                         nb, batch_a, batch_b, batch_c);
      return;
    case 3:
      launch_gemm<3, BF6::BM, BF6::BN, BF6::WM, BF6::WN, BF6::RB, BF6::SWZ, BF6::PF>(
          A, Bt, C, M, N, K, lda, ldb, ldc, accum, st, nb, batch_a, batch_b, batch_c);
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
    gemm_f64(A, Bt, Cpart, M, N, K, lda, ldb, N, false, st, splits, M * N, 1, 0, 0, 0);
}

}  // namespace trg
