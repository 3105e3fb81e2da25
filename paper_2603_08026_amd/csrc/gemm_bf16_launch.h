// bf16 salient-row GEMMs: tile shapes per regime, and what their launchers share.  A launcher to a source file
// (gemm_bf16_raw.hip, gemm_bf16_swiglu.hip, gemm_bf16_down.hip): each holds the paths of its tiles for every
// height, which take a minute to compile.
#pragma once
#include <algorithm>
#include <climits>
#include <cstdlib>
#include "gemm_bf16_dma.h"

namespace dy {

using namespace mm;

namespace {

// Tile shapes per regime (rows = those that exist, or the capacity of a list of up to 128):
//  xlarge  tiles of up to 256 rows x 256 columns (128+128 when gate and up are fused), 2 x 2 waves over
//          the ring loop: a third fewer bytes per flop through the CU's L1 -> LDS path
//          than a 256 x 128 tile and half the LDS operand reads; taken when its coarser tiles still
//          fill the rounds of the chip and every operand can be addressed with 32-bit offsets
//  wide    up to 256 rows x 192 columns (96+96), 4 x 1 waves: 12288 columns are 64 of them, so that few row tiles
//          still make 256 items
//  large   up to 256 rows x 128 columns (64+64), 2 x 2 waves; eight waves over two LDS stages when the operand cannot be
//          addressed that way.  Which of them, how high, how many K splits, and whether a short last row tile
//          goes to the streaming tiles: gemm_plan.h
//  skinny  all rows in one 128-row tile, 64-column tiles, 4 stages in flight and a K split so that
//          about one workgroup per CU streams weights (weight-streaming-bound regime)
//  ONCE: the matrix goes past the L2 where one workgroup alone reads a weight (past_l2)
typedef Shape<256, 256, 2, 2, false, 2> XLargeS;
template <bool ONCE> using XLargeD = Shape<256, 128, 2, 2, true, 2, ONCE>;
template <bool ONCE> using LargeS = Shape<256, 128, 2, 2, false, 2, ONCE>;
template <bool ONCE> using LargeD = Shape<256, 64, 2, 2, true, 2, ONCE>;
typedef Shape<256, 192, 4, 1, false, 2> WideS;
typedef Shape<256, 96, 4, 1, true, 2> WideD;
static_assert(LargeS<false>::BN == 128 && XLargeS::BN == 256 && LargeD<false>::BN == 64 && XLargeD<false>::BN == 128, "columns that the plans count in");
typedef Shape<256, 128, 4, 2, false, 2> LargeS8;  // eight waves, two LDS stages
typedef Shape<256, 64, 4, 2, true, 2> LargeD8;
template <bool ONCE> using SkinnyS = Shape<128, 64, 4, 2, false, 4, ONCE>;
template <bool ONCE> using SkinnyN64 = Shape<128, 64, 4, 1, false, 4, ONCE>;  // the same with four waves, beside the row tiles in one kernel
// skinny regime, wide column tiles (fewer re-reads of the activation tile): q|k|v raw result, and
// gate|up with half-interleaved tiles (48 + 48 or 64 + 64 columns) and SwiGLU in registers
template <bool ONCE> using SkinnyW96 = Shape<128, 96, 4, 1, false, 4, ONCE>;
template <bool ONCE> using SkinnyH128 = Shape<128, 128, 4, 1, false, 4, ONCE>;

// f(std::true_type or std::false_type)
template <typename F> auto with_once(bool once, F f) { return once ? f(std::true_type{}) : f(std::false_type{}); }

int cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
  }
  return n;
}

// The ring loop addresses its operands with a scalar base and 32-bit byte offsets per lane.  The base
// of the activation operand moves with the tile unless rows are gathered: a gathered operand, and
// each weight matrix, must span less than 4 GiB, and a group of permuted weight rows must lie in one matrix;
// otherwise the eight-wave 256 x 128 shapes run.  (Every K split of the plans keeps at least 8
// slices; the loop needs 3.)
// DYLLM_GEMM_NO_RING=1 in the environment takes the fallback for every call (diagnostics and tests).
bool ring_ok(const GemmA &A, int K, const WSeg &seg, int n_rows_w) {
  if (const char *e = getenv("DYLLM_GEMM_NO_RING"))
    if (e[0] == '1') return false;
  const size_t lim = ((size_t)1 << 32) - ((size_t)1 << 20);
  if (A.gather && (A.a_rows == 0 || A.a_rows * (size_t)A.lda * 2 >= lim)) return false;
  if ((size_t)A.lda * 2 * 256 >= lim) return false;
  if ((size_t)n_rows_w * (size_t)K * 2 >= lim) return false;
  if (!ring_groups_ok(seg.n_end[0], seg.n_end[1])) return false;
  return K / BK >= RING_MIN_SLICES;
}

// GEMM of `rows` with one tile shape (host-planned shapes: weight streaming and the eight-wave fallback)
template <typename SH, bool SPLIT, typename Epi>
void run_tiles(const GemmArgs &ga, Epi epi, int splitk, hipStream_t s) {
  // one workgroup per position of the tile order (gemm_tiles) when the list is full, up to 2048 per split
  const int ncol = ga.N / SH::BN, cap = ga.rows.cap;
  const int n_full = (cap / SH::BM) * ncol * splitk, n_part = (cap % SH::BM) ? ncol * splitk : 0;
  int gx = ((n_full + N_XCD - 1) / N_XCD + (n_part + N_XCD - 1) / N_XCD) * N_XCD;
  gx = std::min(std::max(gx, N_XCD), 2048 * splitk);
  set_lds_once<SH, Epi, SPLIT>();
  k_gemm_bf16<SH, Epi, SPLIT><<<gx, SH::NT, SH::LDS_BYTES, s>>>(ga, epi, splitk);
}

int ring_grid() { return std::max(N_XCD, cu_count() / N_XCD * N_XCD); }

int cus_of_xcd() { return ring_grid() / N_XCD; }
bool plan_known(const Rows &rows) { return mm::plan_known(rows.count != nullptr, rows.cap); }
bool wants_plan(Way way, const Rows &rows) { return mm::wants_plan(way, rows.count != nullptr, rows.cap); }
Way way_with(Way way, const Rows &rows, bool made) { return mm::way_with(way, rows.count != nullptr, rows.cap, made); }

constexpr GemmPlan NO_PLAN{0, 1, 0, 1, 256};
// The plan of a GEMM whose row count the host knows; anything else is planned on the device
GemmPlan plan_here(const GemmArgs &ga, const PlanArgs &pa) { return plan_known(ga.rows) ? plan_on_host(pa, ga.rows.cap) : NO_PLAN; }

// GEMM of `rows` in row tiles by a plan: `pl` of plan_here, or the device's in the words of plan_dev, which a row kernel has
// left there (made) or this one leaves
template <typename Kind>
void run_planned(const GemmArgs &ga, typename Kind::Epi epi, const PlanArgs &pa, const GemmPlan &pl, int32_t *plan_dev,
                 bool made, hipStream_t s) {
  const Planned planned = plan_known(ga.rows) ? PLAN_GIVEN : made ? PLAN_MADE : PLAN_HERE;
  set_lds_once_planned<Kind>();
  k_gemm_planned<Kind><<<ring_grid(), 256, RING_SLOTS * RING_SLOT, s>>>(ga, epi, pa, pl, planned, planned == PLAN_GIVEN ? nullptr : plan_dev);
}

// fused: row tiles finish their rows where K is not split
Splits splits_of(const GemmArgs &ga, const GemmPlan &pl, bool fused, const int32_t *plan_dev) {
  Splits sp;
  sp.n = pl.sk;
  sp.tail_from = pl.row_hi;
  sp.n_tail = pl.sk_tail;
  sp.done_to = fused && pl.sk == 1 ? pl.row_hi : 0;
  if (!plan_known(ga.rows)) sp.dev = plan_dev;
  return sp;
}

// q|k|v, out-projection: fp32 result, a row kernel follows
template <typename E, bool ONCE> struct RawKind {
  typedef E Epi;
  typedef XLargeS X;
  typedef LargeS<ONCE> L;
  typedef WideS W;
  static constexpr bool FUSED = false, RAW = true, PLANS = true;
  static __device__ __forceinline__ void stream(const GemmArgs &ga, const Epi &e, int M, int row_lo, int sk, const Walk &w) {
    if (ga.N % SkinnyW96<ONCE>::BN == 0) gemm_tiles<SkinnyW96<ONCE>, EpiStoreF32, true>(ga, e, M, row_lo, INT_MAX, sk, w);
    else gemm_tiles<SkinnyN64<ONCE>, EpiStoreF32, true>(ga, e, M, row_lo, INT_MAX, sk, w);
  }
};

GemmArgs gemm_args(const GemmA &A, const Rows &rows, int K, const WSeg &seg, const void *w2, float *part) {
  return GemmArgs{(const bf16_t *)A.a, A.gather, A.lda, rows, seg.n_end[2], seg, (const bf16_t *)w2, K, part};
}

}  // namespace

}  // namespace dy
