// bf16 down projection with the residual and the scatter in its epilogue, or fp32 sums for a row kernel.
#include "gemm_bf16_launch.h"

namespace dy {

namespace {

template <bool ONCE> struct DownKind {  // residual + scatter in the epilogue, or fp32 sums of a K split
  typedef EpiDown<bf16_t> Epi;
  typedef XLargeS X;
  typedef LargeS<ONCE> L;
  typedef void W;
  static constexpr bool FUSED = true, RAW = true, PLANS = false;
  static __device__ __forceinline__ void stream(const GemmArgs &ga, const Epi &e, int M, int row_lo, int sk, const Walk &w) {
    gemm_tiles<SkinnyN64<ONCE>, Epi, true>(ga, e, M, row_lo, INT_MAX, sk, w);
  }
};

// What the plans of row tiles are made from, and whether a sum kernel follows
struct DownChoice {
  PlanArgs pa;
  bool sums;
};
DownChoice choose_down(const Rows &rows, int N, int K, size_t part_elems) {
  DownChoice c{down_plan_args(N, K, part_elems, true, cus_of_xcd()), true};
  const bool known = plan_known(rows);
  c.sums = known || down_has_sums(c.pa, rows.cap, false);
  if (!c.sums) c.pa.split_ok = c.pa.stream_cols = 0;
  if (known) c.pa.sum_us = 4.0f;
  return c;
}

Way down_way(const Rows &rows, int K, int N) { return way_of(rows.cap, true, ring_ok(GemmA{nullptr, nullptr, K}, K, wseg_one(nullptr, N), N)); }

}  // namespace

PlanJob gemm_bf16_down_plan(Rows rows, int K, int N, size_t part_elems, int32_t *plan_dev) {
  PlanJob job{};
  if (!wants_plan(down_way(rows, K, N), rows)) return job;
  const DownChoice c = choose_down(rows, N, K, part_elems);
  job.make.args = c.pa;
  job.make.rows = rows;
  job.make.words = plan_dev;
  job.sums = c.sums;
  job.make.finishes = true;
  return job;
}

void gemm_bf16_down(GemmA A, Rows rows, int K, int N, const void *wd, const float *h, void *out,
                    float *part, size_t part_elems, const PlanJob &job, hipStream_t s) {
  const Way way = way_with(down_way(rows, K, N), rows, job.make.words);
  if (way == Way::NONE) return;
  const EpiDown<bf16_t> e{h, (bf16_t *)out, N};
  const WSeg seg = wseg_one(wd, N);
  const GemmArgs ga = gemm_args(A, rows, K, seg, nullptr, part);
  PlanArgs pa = down_plan_args(N, K, part_elems, way != Way::EIGHT, cus_of_xcd());
  const bool once = past_l2(N, K);
  Splits sp;
  if (way == Way::STREAM) {
    sp.n = stream_split(pa, rows.cap);
    with_once(once, [&](auto o) {
      if (sp.n == 1) run_tiles<SkinnyS<decltype(o)::value>, false>(ga, e, 1, s);
      else run_tiles<SkinnyS<decltype(o)::value>, true>(ga, e, sp.n, s);
    });
    if (sp.n == 1) return;
  } else if (way == Way::EIGHT) {
    pa.stream_cols = 0;
    sp.n = plan_of(pa, rows.cap, first_on_host(pa, rows.cap)).sk;
    if (sp.n == 1) {
      run_tiles<LargeS8, false>(ga, e, 1, s);
      return;
    }
    run_tiles<LargeS8, true>(ga, e, sp.n, s);
  } else {
    const bool known = plan_known(rows);
    const DownChoice c = known ? choose_down(rows, N, K, part_elems) : DownChoice{job.make.args, job.sums};
    const GemmPlan pl = plan_here(ga, c.pa);
    with_once(once, [&](auto o) { run_planned<DownKind<decltype(o)::value>>(ga, e, c.pa, pl, job.make.words, true, s); });
    if (!c.sums || (known && pl.sk == 1 && pl.row_hi == rows.cap)) return;
    sp = splits_of(ga, pl, true, job.make.words);
  }
  launch_down_finalize(part, sp, h, rows, N, out, s);
}

}  // namespace dy
