// bf16 GEMMs with an fp32 result for a row kernel: q|k|v and the out-projection.
#include "gemm_bf16_launch.h"

namespace dy {

// q|k|v (gemm_bf16_qkv.hip, gemm_bf16_qkv64.hip: heads of 128 and 64 columns), or with an empty QkvOut any raw result
Splits gemm_bf16_qkv128(const GemmArgs &ga, float *part, const QkvOut &out, const PlanArgs &pa, const GemmPlan &pl, int32_t *plan_dev, bool made,
                        hipStream_t s);
Splits gemm_bf16_qkv64(const GemmArgs &ga, float *part, const QkvOut &out, const PlanArgs &pa, const GemmPlan &pl, int32_t *plan_dev, bool made,
                       hipStream_t s);

namespace {

// What a raw result in row tiles is made from: the plan of a full list, and whether the kernel that can finish rows is taken
struct RawChoice {
  PlanArgs pa;
  GemmPlan full;
  bool finishing;
};
// (positions come from a division by at least two, rotary table entries from 32-bit offsets)
bool can_finish(const QkvOut &qkv) { return qkv.tab && qkv.L >= 2 && (size_t)qkv.L * qkv.dh * 4 < ((size_t)1 << 31); }
RawChoice choose_raw(const Rows &rows, int N, int K, size_t part_elems, const QkvOut &qkv) {
  RawChoice c;
  c.pa = raw_plan_args(N, K, part_elems, true, cus_of_xcd());
  const bool known = plan_known(rows);
  const bool few = few_of_room(rows.count != nullptr, rows.cap, qkv.tokens) || few_results(known, rows.cap, (qkv.H + 2 * qkv.Hkv) * qkv.dh) ||
                   (!can_finish(qkv) && qkv.dh == 64);
  c.full = known || !few ? plan_on_host(c.pa, rows.cap) : NO_PLAN;
  c.finishing = finishing_kernel(few, c.full);
  return c;
}

Way raw_way(const GemmA &A, const Rows &rows, int K, const WSeg &seg) { return way_of(rows.cap, true, ring_ok(A, K, seg, seg.n_end[2])); }

}  // namespace

PlanJob gemm_bf16_raw_plan(GemmA A, Rows rows, int K, WSeg seg, size_t part_elems, int32_t *plan_dev, const QkvOut &qkv) {
  PlanJob job{};
  const int N = seg.n_end[2];
  if (!wants_plan(raw_way(A, rows, K, seg), rows)) return job;
  const RawChoice c = choose_raw(rows, N, K, part_elems, qkv);
  job.make.args = c.pa;
  job.full = c.full;
  job.make.rows = rows;
  job.make.words = plan_dev;
  job.finishing = c.finishing;
  job.make.finishes = c.finishing && can_finish(qkv);
  return job;
}

// raw result part[z][j][n], or rows finished as `qkv` says where it has a table; returns the numbers of K splits (on the device if the count is there)
Splits gemm_bf16_raw(GemmA A, Rows rows, int K, WSeg seg, float *part, size_t part_elems, int32_t *plan_dev, const PlanJob &job,
                     const QkvOut &qkv, hipStream_t s) {
  Splits out;
  const Way way = raw_way(A, rows, K, seg);
  if (way == Way::NONE) return out;
  const int N = seg.n_end[2];
  const GemmArgs ga = gemm_args(A, rows, K, seg, nullptr, part);
  PlanArgs pa = raw_plan_args(N, K, part_elems, way != Way::EIGHT, cus_of_xcd());
  const bool once = past_l2(N, K);
  if (way == Way::STREAM) {
    const EpiStoreF32 e{part, N};
    out.n = stream_split(pa, rows.cap);
    with_once(once, [&](auto o) {
      constexpr bool ONCE = decltype(o)::value;
      if (N % SkinnyW96<ONCE>::BN == 0) run_tiles<SkinnyW96<ONCE>, true>(ga, e, out.n, s);
      else run_tiles<SkinnyS<ONCE>, true>(ga, e, out.n, s);
    });
    return out;
  }
  if (way == Way::TILES) {
    const bool made = job.make.words != nullptr, finishes = can_finish(qkv);
    const RawChoice c = made ? RawChoice{job.make.args, job.full, job.finishing} : choose_raw(rows, N, K, part_elems, qkv);
    if (!c.finishing) {
      with_once(once, [&](auto o) {
        run_planned<RawKind<EpiStoreF32, decltype(o)::value>>(ga, EpiStoreF32{part, N}, c.pa, c.full, plan_dev, made, s);
      });
      return splits_of(ga, c.full, false, plan_dev);
    }
    if (finishes && qkv.dh == 64) return gemm_bf16_qkv64(ga, part, qkv, c.pa, c.full, plan_dev, made, s);
    return gemm_bf16_qkv128(ga, part, finishes ? qkv : QkvOut{}, c.pa, c.full, plan_dev, made, s);
  }
  pa.stream_cols = 0;
  out.n = plan_of(pa, rows.cap, first_on_host(pa, rows.cap)).sk;
  run_tiles<LargeS8, true>(ga, EpiStoreF32{part, N}, out.n, s);
  return out;
}

}  // namespace dy
