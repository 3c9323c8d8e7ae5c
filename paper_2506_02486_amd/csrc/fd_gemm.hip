// fd_gemm.hip -- the local block product of Cannon's matrix multiply on gfx950.
//
// In Cannon's algorithm each of P ranks holds row stripes of Ns = N/P rows and, at
// each of its P steps, multiplies an Ns x Ns block of its A stripe with the B
// stripe it holds, adding the N * Ns * Ns multiply-adds into its C stripe
// (Sec. 4.4).  That step is C = C + A B, a dense contraction, so it runs on the
// FP64 matrix cores (v_mfma_f64_16x16x4f64): the paper states no element type,
// and FP64 is the precision of the oracle that defines the product.
//
// Large products (gemm_f64_kernel).  Block: 1024 threads (16 waves), a 256 x 128 tile
// of C; each wave owns a 32 x 64 piece as 2 x 4 MFMA tiles of 16 x 16 (8 independent
// accumulators of 4 doubles per lane), so that four waves share each SIMD.  The K loop
// takes 16 columns of A and 16 rows of B per stage, staged in double-buffered LDS.  The
// matrix cores bound it, and what kept them idle was that all waves of the block wrote a
// stage to LDS, met at the barrier and read their first fragments at the same time
// (MFMA utilisation 84.7%), so the non-MFMA work is spread between the MFMAs:
//   * a stage is written to LDS in the middle of the MFMAs of the stage before it,
//     from registers loaded one whole stage earlier;
//   * fragments are double-buffered: each k-step's are read during the MFMAs of the
//     one before, and the last k-step's MFMAs run after the barrier, while the first
//     fragments of the next stage arrive;
//   * LDS accesses and loads are issued one MFMA at a time (sched_group_barrier).
//   * the loop takes two stages a turn, so that the LDS buffer is known when compiling
//     and no address is computed between the barrier and the reads behind it.
// 3780 x 30240 x 3780: 65.3 -> 69.1 TFLOP/s (67.4 with the buffer chosen at run time);
// 8192^3: 68.2 -> 70.3-71.0 before that (vendor BLAS 72.1 on the same box).  Writing a
// stage earlier alone gave nothing (64.4), with the double fragments 67.4.
//
// Smaller products (gemm_pair_kernel) leave most CUs idle with 256 x 128 tiles (512 x
// 4096 x 512, one of Cannon's products at N = 4096 and P = 8: 64 tiles on 256 CUs), so
// they take 128 x 128, 64 x 64, 32 x 64 or 32 x 32 tiles, whichever the cost model below
// (gemm_tile) prices lowest.  Their waves own 32 x 32, 16 x 32 or 16 x 16 pieces, for
// which fragment reads of single doubles would bound the kernel (58 of LDS's 128 bytes
// per clock at 64 x 64, as 8-byte reads): K is kept in pairs in LDS (A [m][k], B [k/2][n]
// [2]) and a lane reads two k-steps with one 16-byte access, step h of a pair taking k =
// 8 p + 2 (lane / 16) + h (any order of k will do as long as A and B agree).  The
// elements of C to add to are read before the K loop.  Same pipelining otherwise.
// Measured (us, before / after; before: 256 x 128 tiles): 512 x 4096 x 512 140 / 40.7
// (52.7 TFLOP/s), 1000 x 4000 x 1000 260 / 134, 1285 x 7710 x 1285 662 / 447, 700^3 184 /
// 18.3, 256 x 2048 x 256 72 / 8.8, 52 x 260 x 52 26 / 7.7 (the launch rate of the loop
// that timed it).
//
// The products of one rank (fd_cannon_rank_f64) in one launch (PARTS), where the tiles are 64
// x 64 or smaller: a block takes its tile through all of them, the loads of the next
// product's first stage issued during the last stages of the one before, and adds each
// to the C it holds in registers, so the bits are those of the separate products.
// Separately, each of them starts with an empty pipeline, ends with a last wave of tiles
// and reads and writes C, and small ones are over before the next is launched (us, P
// launches / one): 8 x 32 x 256 x 32 91 / 9.2, 8 x 135 x 1080 x 135 91 / 24, 4 x 446 x
// 1784 x 446 84.8 / 75.0, 8 x 512 x 4096 x 512 325 / 278, 5 x 927 x 4635 x 927 795 / 753.
// The larger tiles have no registers for the sum beside the accumulators (128 x 128: 617
// against 606 separately at 6 x 736 x 4416 x 736).
//
// Operands of any shape and leading dimension: K is split into a first stage of 1 to a
// whole stage's columns, whose loads past K read 0, and whole stages, whose loads need no
// bounds arithmetic (an offset per thread from the tile's base plus the stage's offset);
// rows past m and columns past n are read clamped and their results not stored.  Blocks
// sharing a B panel (a column of tiles) run on one XCD in succession, so that the panel
// is read from HBM about once.
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fd.h"
#include "fd_internal.h"

namespace fd {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
// two consecutive doubles in memory, aligned as one
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

constexpr int BM = 256;          // tile rows (M)
constexpr int BN = 128;          // tile columns (N)
constexpr int BK = 16;           // K per stage
constexpr int WTM = 32;          // wave tile rows
constexpr int WTN = 64;          // wave tile columns
constexpr int WAVES_N = BN / WTN;
constexpr int GT = 64 * (BM / WTM) * WAVES_N;  // threads per block
constexpr int FM = WTM / 16;     // MFMA tiles per wave, rows
constexpr int FN = WTN / 16;     // MFMA tiles per wave, columns
// LDS pitches (doubles), chosen so that the 64 lanes of a fragment read (16 rows or
// columns x 4 k) fall on distinct banks in each half-wave: A is kept row-major [m][k]
// with pitch 18 (36 fr + 2 fk distinct mod 64 dwords), B as [k][n] with pitch 144
// (consecutive k 32 banks apart).
constexpr int SA = BK + 2;
constexpr int SB = BN + 16;
// waves per SIMD the register budget must allow (the second __launch_bounds__
// argument): one block of 16 waves per CU (LDS 110.6 KB of 160 KB), at most 128
// VGPRs per lane
constexpr int WAVES_PER_SIMD = 4;
constexpr int A_PER = BM * BK / GT;  // A elements a thread loads per stage
constexpr int B_PER = BK * BN / GT;  // B elements a thread loads per stage

struct GemmArgs {
  int64_t m, n, k;
  const double* a;
  int64_t lda;
  const double* b;
  int64_t ldb;
  double* c;
  int64_t ldc;
  int tiles_m;
  int accumulate;
  // PARTS: k is one part of K; part q is columns q k .. of A and rows q k .. of B, and
  // the products of all of them, from part `first` on and around, are added to C one
  // after the other (k >= 32, accumulate)
  int parts, first;
};

// The stages of all parts in order: the addresses of the one to load next, kept ready so
// that its loads wait for no arithmetic.  They are consecutive columns of A and rows of B
// but where the last part is followed by part 0; past the last stage they stay.
struct Stages {
  const double *a, *b;  // of the next stage
  int lim;              // its columns that count: kt in a part's first stage, else bk
  int kt, bk, per;      // per: stages of a part
  int s, part, left;    // stage within the part, part, stages after this one
  __device__ __forceinline__ void step(const GemmArgs& g) {
    if (left == 0) return;
    --left;
    a += lim;
    b += lim * g.ldb;
    const bool next = ++s == per;
    s = next ? 0 : s;
    part += next ? 1 : 0;
    if (part == g.parts) {
      part = 0;
      a -= g.parts * g.k;
      b -= g.parts * g.k * g.ldb;
    }
    lim = next ? kt : bk;
  }
};

// Which of the two LDS buffers a stage is in, known when compiling (loops take two stages a
// turn), so that no address is computed between the barrier and the reads behind it.
template <int B>
using Parity = std::integral_constant<int, B>;

// Blocks b, b+8, b+16, ... run on one XCD; give each XCD a contiguous run of
// logical tiles (row tiles fastest: the tiles of one B panel).
__device__ __forceinline__ int remap_gemm(int bid, int nb) {
  const int per = nb >> 3;
  if (bid < (per << 3)) return (bid & 7) * per + (bid >> 3);
  return bid;
}

// OFF: the type of an element's offset from its tile's base: 32 bits, or 64 where a
// leading dimension is too large for that (gemm_offsets_fit).
template <class OFF>
__global__ void __launch_bounds__(GT, WAVES_PER_SIMD) gemm_f64_kernel(GemmArgs g) {
  __shared__ double sa[2][BM * SA];
  __shared__ double sb[2][BK * SB];

  const int logical = remap_gemm(blockIdx.x, gridDim.x);
  const int64_t m0 = (int64_t)(logical % g.tiles_m) * BM;
  const int64_t n0 = (int64_t)(logical / g.tiles_m) * BN;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = t >> 6;
  const int wm = (w / WAVES_N) * WTM;
  const int wn = (w % WAVES_N) * WTN;

  // stage loads: A as BK consecutive k of rows t / BK + (GT / BK) i; B as BN
  // consecutive columns of rows t / BN + (GT / BN) i (each instruction: 4 rows of 128
  // bytes of A, 512 contiguous bytes of B)
  const int ak = t % BK;
  const int ar = t / BK;
  const int bc = t % BN;
  const int br = t / BN;
  // K is taken as a first stage of kt = k - (stages - 1) BK columns (1..BK), then
  // whole stages of BK.  Rows of A past m and columns of B past n are read clamped and
  // not cleared: they only reach rows and columns of the tile that are not stored.
  // Only the first stage clears what lies past its kt columns (in both operands: 0 x
  // Inf would be NaN).  So a load of a whole stage is a per-thread offset from the
  // stage's uniform base, with no bounds arithmetic, and every load is unconditional
  // (a load under a branch would make the compiler wait for it where the branch joins).
  const int64_t stages = (g.k + BK - 1) / BK;
  const int64_t kt = g.k - (stages - 1) * BK;
  const double* At = g.a + m0 * g.lda;
  const double* Bt = g.b + n0;
  const int mr = (int)std::min<int64_t>(g.m - m0, BM) - 1;  // last row and column of C
  const int nr = (int)std::min<int64_t>(g.n - n0, BN) - 1;  // in the tile
  OFF oa[A_PER], ob[B_PER];
#pragma unroll
  for (int i = 0; i < A_PER; ++i)  // (k < BK: a single stage, read clamped in K)
    oa[i] = (OFF)std::min(ar + (GT / BK) * i, mr) * (OFF)g.lda +
            (OFF)std::min<int64_t>(ak, g.k - 1);
#pragma unroll
  for (int i = 0; i < B_PER; ++i)
    ob[i] = (OFF)std::min<int64_t>(br + (GT / BN) * i, g.k - 1) * (OFF)g.ldb +
            (OFF)std::min(bc, nr);
  double ra[A_PER], rb[B_PER];
  // whole stage s >= 1 at column k0 = kt + (s - 1) BK of A, row k0 of B (past the last
  // stage: that one again, into the buffer nobody reads)
  auto load_stage = [&](int64_t s) {
    const int64_t k0 = std::max<int64_t>(kt + (std::min(s, stages - 1) - 1) * BK, 0);
    const double* Ak = At + k0;
    const double* Bk = Bt + k0 * g.ldb;
#pragma unroll
    for (int i = 0; i < A_PER; ++i) ra[i] = Ak[oa[i]];
#pragma unroll
    for (int i = 0; i < B_PER; ++i) rb[i] = Bk[ob[i]];
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < A_PER; ++i) sa[buf][(ar + (GT / BK) * i) * SA + ak] = ra[i];
#pragma unroll
    for (int i = 0; i < B_PER; ++i) sb[buf][(br + (GT / BN) * i) * SB + bc] = rb[i];
  };

  d4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  if (stages > 0) {
    // the first stage: columns 0 .. kt-1 of A and rows 0 .. kt-1 of B, the rest 0
    // (a cleared element reads the stage's last valid one, in bounds)
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      const double x = At[(int64_t)std::min(ar + (GT / BK) * i, mr) * g.lda +
                          std::min<int64_t>(ak, kt - 1)];
      ra[i] = ak < kt ? x : 0.0;
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
      const int64_t row = br + (GT / BN) * i;
      const double x = Bt[std::min(row, kt - 1) * g.ldb + std::min(bc, nr)];
      rb[i] = row < kt ? x : 0.0;
    }
    store_stage(0);
    load_stage(1);
  }
  __syncthreads();
  // fragment lanes: A rows / B columns lane % 16 of a 16-wide tile, k = lane / 16
  const int fr = lane & 15;
  const int fk = lane >> 4;
  const int fa = (wm + fr) * SA + fk;
  const int fb = fk * SB + wn + fr;
  double af[2][FM], bf[2][FN];
  auto frags = [&](int set, int buf, int kk) {
#pragma unroll
    for (int i = 0; i < FM; ++i) af[set][i] = sa[buf][fa + 16 * i * SA + kk];
#pragma unroll
    for (int j = 0; j < FN; ++j) bf[set][j] = sb[buf][fb + kk * SB + 16 * j];
  };
  constexpr int NQ = BK / 4;
  static_assert(NQ % 2 == 0, "the fragment sets alternate over a stage");
  frags(0, 0, 0);
  auto stage = [&](auto parity, int64_t s) {
    constexpr int buf = decltype(parity)::value;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      __builtin_amdgcn_sched_barrier(0);
      // the next k-step's fragments; those of the next stage after the barrier, past
      // which nobody reads this stage's buffer any more
      if (q < NQ - 1) {
        frags((q + 1) & 1, buf, 4 * (q + 1));
      } else {
        __syncthreads();
        frags(0, buf ^ 1, 0);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[q & 1][i], bf[q & 1][j], acc[i][j],
                                                           0, 0, 0);
      if (q == 0) {
        store_stage(buf ^ 1);
        load_stage(s + 2);
      }
      // issue order: one MFMA (0x8), then its share of the LDS reads (0x100) and, in
      // the first k-step, of the LDS writes (0x200) and loads (0x20)
      constexpr int NM = FM * FN, NR = FM + FN, NW = A_PER + B_PER;
      static_assert(NR <= NM && NW <= NM, "at most one of each per MFMA");
#pragma unroll
      for (int z = 0; z < NM; ++z) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        if ((z + 1) * NR / NM != z * NR / NM) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (q == 0 && (z + 1) * NW / NM != z * NW / NM) {
          __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
        }
      }
    }
  };
  int64_t s = 0;
  for (; s + 1 < stages; s += 2) {
    stage(Parity<0>(), s);
    stage(Parity<1>(), s + 1);
  }
  if (s < stages) stage(Parity<0>(), s);

  // accumulator element v of lane l holds row l / 16 + 4 v, column l % 16 of its
  // 16 x 16 tile (the lane layout of v_mfma_f64_16x16x4f64, checked with one-hot
  // operands on the device)
  int tt = t;
  asm volatile("" : "+v"(tt));  // keeps these addresses out of the loop's registers
  const int r0 = (tt >> 6) / WAVES_N * WTM + ((tt & 63) >> 4);
  const int c0 = (tt >> 6) % WAVES_N * WTN + (tt & 15);
  double* const ct = g.c + (m0 + r0) * g.ldc + n0 + c0;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double* const p = ct + (16 * i + 4 * v) * g.ldc;
#pragma unroll
      for (int j = 0; j < FN; ++j)
        if (r0 + 16 * i + 4 * v <= mr && c0 + 16 * j <= nr)
          p[16 * j] = g.accumulate ? p[16 * j] + acc[i][j][v] : acc[i][j][v];
    }
}

// Tiles of PM x PN of waves of VM x VN, stages of PK columns; at most 16 waves per CU
// (four per SIMD) in the register budget.
template <int PM, int PN, int VM, int VN, int PK, bool PARTS>
__global__ void __launch_bounds__(64 * (PM / VM) * (PN / VN), WAVES_PER_SIMD)
    gemm_pair_kernel(GemmArgs g) {
  constexpr int WN = PN / VN;
  constexpr int PT = 64 * (PM / VM) * WN;  // threads
  constexpr int FI = VM / 16, FJ = VN / 16;
  constexpr int KP = PK / 2;   // pairs of k per stage
  constexpr int PA = PK + 2;   // LDS pitches: A row, B pair row (16-byte reads of 8 lanes
  constexpr int PB = 2 * PN;   // fall on distinct banks)
  constexpr int NA = PM * KP / PT, NB = KP * PN / PT;  // pairs a thread loads per stage
  constexpr int NP = PK / 8;   // pairs of k-steps per stage
  static_assert(NA * PT == PM * KP && NB * PT == KP * PN && NP % 2 == 0, "tile shape");
  __shared__ __attribute__((aligned(16))) double sa[2][PM * PA];
  __shared__ __attribute__((aligned(16))) double sb[2][KP * PB];

  const int logical = remap_gemm(blockIdx.x, gridDim.x);
  const int64_t m0 = (int64_t)(logical % g.tiles_m) * PM;
  const int64_t n0 = (int64_t)(logical / g.tiles_m) * PN;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wm = (w / WN) * VM, wn = (w % WN) * VN;
  const int64_t stages = (g.k + PK - 1) / PK;  // k >= 1
  const int64_t kt = g.k - (stages - 1) * PK;
  const int64_t all = PARTS ? stages * g.parts : stages;
  const double* At = g.a + m0 * g.lda;
  const double* Bt = g.b + n0;
  if (PARTS) {
    At += g.first * g.k;
    Bt += g.first * g.k * g.ldb;
  }
  Stages st{At, Bt, (int)kt, (int)kt, PK, (int)stages, 0, g.first, (int)stages * g.parts - 1};
  if (PARTS) st.step(g);  // (the first is loaded below)
  int lim = PK;  // columns of the stage in ra and rb that count
  const int mr = (int)std::min<int64_t>(g.m - m0, PM) - 1;
  const int nr = (int)std::min<int64_t>(g.n - n0, PN) - 1;
  // thread's pair i of A: row e / KP, pair e % KP; of B: pair row e / PN, column e % PN
  unsigned oa[NA], ob[NB];
  int la[NA], lb[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int e = t + PT * i, row = e / KP, kp = e % KP;
    oa[i] = (unsigned)std::min(row, mr) * (unsigned)g.lda + 2u * kp;
    la[i] = row * PA + 2 * kp;
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int e = t + PT * i, kp = e / PN, col = e % PN;
    ob[i] = 2u * kp * (unsigned)g.ldb + (unsigned)std::min(col, nr);
    lb[i] = kp * PB + 2 * col;
  }
  d2 ra[NA], rb[NB];
  auto load_stage = [&](int64_t s) {  // whole stage 1 <= s < stages
    const int64_t k0 = kt + (s - 1) * PK;
    const double* Ak = PARTS ? st.a : At + k0;
    const double* Bk = PARTS ? st.b : Bt + k0 * g.ldb;
    lim = st.lim;
#pragma unroll
    for (int i = 0; i < NA; ++i) ra[i] = *reinterpret_cast<const d2u*>(Ak + oa[i]);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      rb[i][0] = Bk[ob[i]];
      rb[i][1] = (Bk + g.ldb)[ob[i]];
    }
    if (PARTS) st.step(g);
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NA; ++i) *reinterpret_cast<d2*>(&sa[buf][la[i]]) = ra[i];
#pragma unroll
    for (int i = 0; i < NB; ++i) *reinterpret_cast<d2*>(&sb[buf][lb[i]]) = rb[i];
  };
  // the first stage: kt columns of A and rows of B, the rest 0
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int e = t + PT * i;
    const double* row = At + (int64_t)std::min(e / KP, mr) * g.lda;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t k = 2 * (e % KP) + h;
      const double x = row[std::min(k, kt - 1)];
      ra[i][h] = k < kt ? x : 0.0;
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int e = t + PT * i;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t k = 2 * (e / PN) + h;
      const double x = Bt[std::min(k, kt - 1) * g.ldb + std::min(e % PN, nr)];
      rb[i][h] = k < kt ? x : 0.0;
    }
  }
  const int fr = lane & 15, fk = lane >> 4;
  // C to add to (an element outside C reads the tile's last row or column)
  double c0[FI][FJ][4];  // (set and used where g.accumulate)
  if (g.accumulate) {
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int j = 0; j < FJ; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          c0[i][j][v] = g.c[(m0 + std::min(wm + 16 * i + fk + 4 * v, mr)) * g.ldc + n0 +
                            std::min(wn + 16 * j + fr, nr)];
  }
  d4 acc[FI][FJ];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  store_stage(0);
  if (all > 1) load_stage(1);
  __syncthreads();
  // fragments of a pair of k-steps: lane l holds k = 8 p + 2 (l / 16) + {0, 1} of row /
  // column l % 16
  const int fa = (wm + fr) * PA + 2 * fk, fb = fk * PB + 2 * (wn + fr);
  d2 af[2][FI], bf[2][FJ];
  auto frags = [&](int set, int buf, int p) {
#pragma unroll
    for (int i = 0; i < FI; ++i)
      af[set][i] = *reinterpret_cast<const d2*>(&sa[buf][fa + 16 * i * PA + 8 * p]);
#pragma unroll
    for (int j = 0; j < FJ; ++j)
      bf[set][j] = *reinterpret_cast<const d2*>(&sb[buf][fb + 4 * p * PB + 32 * j]);
  };
  auto mma = [&](int set) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < FI; ++i)
#pragma unroll
        for (int j = 0; j < FJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[set][i][h], bf[set][j][h],
                                                           acc[i][j], 0, 0, 0);
  };
  frags(0, 0, 0);
  int64_t last = stages - 1;  // PARTS: the current part's last stage
  for (int64_t s = 0; s + 1 < all; ++s) {
    const int buf = (int)(s & 1);
    if (PARTS && lim < PK) {  // a part's first stage is to be stored: clear its rest
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < NA; ++i) ra[i][h] = 2 * ((t + PT * i) % KP) + h < lim ? ra[i][h] : 0.0;
#pragma unroll
        for (int i = 0; i < NB; ++i) rb[i][h] = 2 * ((t + PT * i) / PN) + h < lim ? rb[i][h] : 0.0;
      }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      __builtin_amdgcn_sched_barrier(0);
      if (q < NP - 1) {
        frags((q + 1) & 1, buf, q + 1);
      } else {  // past the barrier nobody reads this stage's buffer any more
        __syncthreads();
        frags(0, buf ^ 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      mma(q & 1);
      if (q == 0) {
        __builtin_amdgcn_sched_barrier(0);
        store_stage(buf ^ 1);
        load_stage(std::min(s + 2, stages - 1));
      }
    }
    if (PARTS && s == last) {
      last += stages;
#pragma unroll
      for (int i = 0; i < FI; ++i)
#pragma unroll
        for (int j = 0; j < FJ; ++j) {
#pragma unroll
          for (int v = 0; v < 4; ++v) c0[i][j][v] += acc[i][j][v];
          acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
        }
    }
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    if (q < NP - 1) frags((q + 1) & 1, (int)((all - 1) & 1), q + 1);
    mma(q & 1);
  }
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j) {
      const int col = wn + 16 * j + fr;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wm + 16 * i + fk + 4 * v;
        if (row <= mr && col <= nr) {
          double* p = g.c + (m0 + row) * g.ldc + n0 + col;
          *p = g.accumulate ? c0[i][j][v] + acc[i][j][v] : acc[i][j][v];
        }
      }
    }
}

// The tile shapes, largest first.
struct TileCost {
  int m, n;
  double busy;   // us a CU spends on one tile per 16 of K when it has several
  double alone;  // the same for the last one, which shares its CU with no other
};
// From 2048 x 8192 x 2048 (every CU has several tiles) and, alone, from products with one
// tile per CU (1000 x 4000 x 1000, 256 x 2048 x 256) or fewer.
constexpr TileCost kTiles[5] = {{256, 128, 3.86, 3.90},
                                {128, 128, 2.04, 2.09},
                                {64, 64, 0.552, 0.69},
                                {32, 64, 0.302, 0.40},
                                {32, 32, 0.14, 0.29}};

// The tile shape of least modelled time: the fullest CU's tiles, one after the other.
// The model is within 8% of the measured time of every shape on 512 x 4096 x 512, 972 x 7776
// x 972, 1285 x 7710 x 1285, 1875 x 7500 x 1875, 2048 x 8192 x 2048 and 3780 x 30240 x
// 3780, so its choice is the fastest or as good (us with 256 x 128, 128 x 128 and 64 x 64):
// 132 / 72 / 41, 245 / 263 / 269, 621 / 507 / 450, 907 / 966 / 913, 994 / 1059 / 1127 and
// 12502 / 13342 / 14570.  Small ones with 64 x 64, 32 x 64 and 32 x 32 (us a rank's products
// at N / P): 516 / 4 26.5 / 17.7 / 13.5, 1080 / 8 49 / 32.1 / 24.4, 1124 / 4 (324 tiles of 32 x
// 32) 49 / 29.1 / 31.3, 2000 / 8 84 / 49.7 / 53.5, 1784 / 4 75.1 / 70.8 / 76.6.
int gemm_tile(int64_t m, int64_t n) {
  int best = 0;
  double cost = -1.0;
  for (int i = 0; i < 5; ++i) {
    const double tiles = (double)((m + kTiles[i].m - 1) / kTiles[i].m) *
                         (double)((n + kTiles[i].n - 1) / kTiles[i].n);
    const double most = std::ceil(tiles / 256.0);
    const double c = (most - 1.0) * kTiles[i].busy + kTiles[i].alone;
    if (cost < 0.0 || c < cost) {
      cost = c;
      best = i;
    }
  }
  return best;
}

// Tiles up to which all products of a rank go in one launch: 1095 (5 x 927 x 4635 x 927) 753
// us against 795, 1683 (6 x 1051 x 6306 x 1051) 1536 / 1546, 3100 (5 x 1582 x 7910 x 1582)
// 3655 / 3498.
constexpr int64_t kPartsTiles = 2048;

bool one_launch_pays(int64_t m, int64_t n) {
  const int tile = gemm_tile(m, n);
  const int64_t tiles = (m + kTiles[tile].m - 1) / kTiles[tile].m *
                        ((n + kTiles[tile].n - 1) / kTiles[tile].n);
  return tile >= 2 && tiles <= kPartsTiles;
}

// Offsets from a tile's base fit 32 bits: at most 256 rows of A or 32 of B.
bool gemm_offsets_fit(int64_t lda, int64_t ldb) { return lda < (1LL << 23) && ldb < (1LL << 26); }

// Last byte (exclusive) a row-major rows x cols operand with leading dimension ld
// occupies, from its first element.
int64_t extent_bytes(int64_t rows, int64_t cols, int64_t ld) {
  if (rows <= 0 || cols <= 0) return 0;
  return 8 * ((rows - 1) * ld + cols);
}

bool ranges_overlap(const void* p, int64_t pn, const void* q, int64_t qn) {
  if (pn <= 0 || qn <= 0) return false;
  const char* a = static_cast<const char*>(p);
  const char* b = static_cast<const char*>(q);
  return a < b + qn && b < a + pn;
}

}  // namespace
}  // namespace fd

using namespace fd;

namespace {

// The argument checks of one product, in its own name.
int gemm_checked(int64_t m, int64_t n, int64_t k, const double* a, int64_t lda, const double* b,
                 int64_t ldb, const double* c, int64_t ldc, const char* who) {
  if (!c) return fail(FD_EINVAL, "%s: c is NULL", who);
  if (ldc < n) return fail(FD_EINVAL, "%s: ldc < n", who);
  if (k > 0) {
    if (!a || !b) return fail(FD_EINVAL, "%s: a or b is NULL", who);
    if (lda < k || ldb < n) return fail(FD_EINVAL, "%s: lda < k or ldb < n", who);
    const int64_t cb = extent_bytes(m, n, ldc);
    if (ranges_overlap(c, cb, a, extent_bytes(m, k, lda)) ||
        ranges_overlap(c, cb, b, extent_bytes(k, n, ldb)))
      return fail(FD_EINVAL, "%s: c overlaps a or b", who);
  }
  return FD_OK;
}

// parts of k columns each, from part `first` on (parts == 1: one product)
int gemm_run(int64_t m, int64_t n, int64_t k, int parts, int first, const double* a, int64_t lda,
             const double* b, int64_t ldb, double* c, int64_t ldc, int accumulate,
             hipStream_t s, const char* who) {
  // (k == 0 only clears or keeps C, and large leading dimensions need 64-bit offsets:
  // both by the first kernel)
  const bool fits = gemm_offsets_fit(lda, ldb);
  const int tile = k > 0 && fits ? gemm_tile(m, n) : 0;
  const int64_t tm = (m + kTiles[tile].m - 1) / kTiles[tile].m;
  const int64_t tn = (n + kTiles[tile].n - 1) / kTiles[tile].n;
  if (tm * tn > 0x7fffffffLL || tm > 0x7fffffffLL) return fail(FD_EINVAL, "%s: too many tiles", who);
  const GemmArgs g{m, n, k, a, lda, b, ldb, c, ldc, (int)tm, accumulate, parts, first};
  const dim3 grid((unsigned)(tm * tn));
  void (*kernel)(GemmArgs) = fits ? gemm_f64_kernel<unsigned> : gemm_f64_kernel<int64_t>;
  int threads = GT;
  if (tile == 1) {
    kernel = gemm_pair_kernel<128, 128, 32, 32, 16, false>;
    threads = 1024;
  } else if (tile == 2) {
    kernel = parts > 1 ? gemm_pair_kernel<64, 64, 16, 32, 16, true>
                       : gemm_pair_kernel<64, 64, 16, 32, 16, false>;
    threads = 512;
  } else if (tile == 3) {
    kernel = parts > 1 ? gemm_pair_kernel<32, 64, 16, 16, 32, true>
                       : gemm_pair_kernel<32, 64, 16, 16, 32, false>;
    threads = 512;
  } else if (tile == 4) {
    kernel = parts > 1 ? gemm_pair_kernel<32, 32, 16, 16, 32, true>
                       : gemm_pair_kernel<32, 32, 16, 16, 32, false>;
    threads = 256;
  }
  hipLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), 0, s, g);
  return check_hip(hipGetLastError(), who);
}

}  // namespace

extern "C" int fd_block_gemm_f64(int64_t m, int64_t n, int64_t k, const double* a, int64_t lda,
                                 const double* b, int64_t ldb, double* c, int64_t ldc,
                                 int32_t accumulate, void* stream) {
  if (m < 0 || n < 0 || k < 0) return fail(FD_EINVAL, "fd_block_gemm_f64: negative extent");
  if (m == 0 || n == 0) return FD_OK;
  const int rc = gemm_checked(m, n, k, a, lda, b, ldb, c, ldc, "fd_block_gemm_f64");
  if (rc) return rc;
  return gemm_run(m, n, k, 1, 0, a, lda, b, ldb, c, ldc, accumulate ? 1 : 0,
                  reinterpret_cast<hipStream_t>(stream), "fd_block_gemm_f64");
}

extern "C" int fd_cannon_rank_f64(int64_t n, int32_t parts, int32_t rank, const double* a,
                                  int64_t lda, const double* b, int64_t ldb, double* c,
                                  int64_t ldc, void* stream) {
  const char* who = "fd_cannon_rank_f64";
  if (n < 0 || parts < 1 || n % parts) return fail(FD_EINVAL, "%s: n is not P stripes", who);
  const int64_t ns = n / parts;
  if (ns == 0) return FD_OK;
  const int first = (int)(((int64_t)rank % parts + parts) % parts);
  for (int i = 0; i < parts; ++i) {
    const int q = (first + i) % parts;
    const int rc = gemm_checked(ns, n, ns, a ? a + q * ns : a, lda, b ? b + q * ns * ldb : b, ldb,
                                c, ldc, who);
    if (rc) return rc;
  }
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  // one launch for all products in tiles of 64 x 64 and less, from ns = 32 on (a part's
  // first stage is read whole) and up to kPartsTiles: with more tiles, blocks in
  // different parts of K share less of the B panels in L2
  if (ns >= 32 && gemm_offsets_fit(lda, ldb) && one_launch_pays(ns, n))
    return gemm_run(ns, n, ns, parts, first, a, lda, b, ldb, c, ldc, 1, s, who);
  for (int i = 0; i < parts; ++i) {
    const int q = (first + i) % parts;
    const int rc = gemm_run(ns, n, ns, 1, 0, a + q * ns, lda, b + q * ns * ldb, ldb, c, ldc, 1, s,
                            who);
    if (rc) return rc;
  }
  return FD_OK;
}
