// bf16 gate|up GEMM with SwiGLU in its epilogue.
#include "gemm_bf16_launch.h"

namespace dy {

namespace {

// weight streaming of gate|up: tiles of HALF gate + HALF up columns, SwiGLU in registers, no raw result
// (the FFN width is a multiple of 64 for every bf16 configuration the library accepts)
__host__ __device__ __forceinline__ GemmArgs halves_args(const GemmArgs &ga) {
  GemmArgs h = ga;
  h.seg.w[1] = h.seg.w[2] = ga.W2;
  h.seg.n_end[0] = ga.N;
  h.seg.n_end[1] = h.seg.n_end[2] = 2 * ga.N;
  h.N = 2 * ga.N;
  return h;
}
template <bool ONCE> struct SwigluKind {
  typedef EpiSwiGLU<bf16_t> Epi;
  typedef XLargeD<ONCE> X;
  typedef LargeD<ONCE> L;
  typedef WideD W;
  static constexpr bool FUSED = true, RAW = false, PLANS = false;
  static __device__ __forceinline__ void stream(const GemmArgs &ga, const Epi &e, int M, int row_lo, int, const Walk &w) {
    const GemmArgs h = halves_args(ga);
    if (ga.N % 48 == 0) gemm_tiles<SkinnyW96<ONCE>, EpiSwiGLUHalves<bf16_t, 48>, false>(h, EpiSwiGLUHalves<bf16_t, 48>{e.act, ga.N}, M, row_lo, INT_MAX, 1, w);
    else gemm_tiles<SkinnyH128<ONCE>, EpiSwiGLUHalves<bf16_t, 64>, false>(h, EpiSwiGLUHalves<bf16_t, 64>{e.act, ga.N}, M, row_lo, INT_MAX, 1, w);
  }
};

Way swiglu_way(const Rows &rows, int K, int N) {
  return way_of(rows.cap, N % 48 == 0 || N % 64 == 0, ring_ok(GemmA{nullptr, nullptr, K}, K, wseg_one(nullptr, N), N));
}

}  // namespace

PlanJob gemm_bf16_swiglu_plan(Rows rows, int K, int N, int32_t *plan_dev) {
  PlanJob job{};
  if (!wants_plan(swiglu_way(rows, K, N), rows)) return job;
  job.make.args = swiglu_plan_args(N, K, cus_of_xcd());
  job.make.rows = rows;
  job.make.words = plan_dev;
  return job;
}

void gemm_bf16_swiglu(GemmA A, Rows rows, int K, int N, const void *wg, const void *wu, void *act, const PlanJob &job, hipStream_t s) {
  const Way way = way_with(swiglu_way(rows, K, N), rows, job.make.words);
  if (way == Way::NONE) return;
  const EpiSwiGLU<bf16_t> e{(bf16_t *)act, N};
  const WSeg seg = wseg_one(wg, N);
  const GemmArgs ga = gemm_args(A, rows, K, seg, wu, nullptr);
  const bool once = past_l2(2 * N, K);
  if (way == Way::STREAM) {
    with_once(once, [&](auto o) {
      constexpr bool ONCE = decltype(o)::value;
      if (N % 48 == 0) run_tiles<SkinnyW96<ONCE>, false>(halves_args(ga), EpiSwiGLUHalves<bf16_t, 48>{(bf16_t *)act, N}, 1, s);
      else run_tiles<SkinnyH128<ONCE>, false>(halves_args(ga), EpiSwiGLUHalves<bf16_t, 64>{(bf16_t *)act, N}, 1, s);
    });
  } else if (way == Way::EIGHT) {
    run_tiles<LargeD8, false>(ga, e, 1, s);
  } else {
    const PlanArgs pa = swiglu_plan_args(N, K, cus_of_xcd());
    with_once(once, [&](auto o) { run_planned<SwigluKind<decltype(o)::value>>(ga, e, pa, plan_here(ga, pa), job.make.words, true, s); });
  }
}

}  // namespace dy
