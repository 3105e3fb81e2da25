// bf16 GEMMs with an fp32 result for a row kernel: q|k|v and the out-projection.
#include "gemm_bf16_launch.h"

namespace dy {

namespace {

struct RawKind {  // q|k|v, out-projection: fp32 result, a row kernel follows
  typedef EpiStoreF32 Epi;
  typedef XLargeS X;
  typedef LargeS L;
  typedef WideS W;
  static constexpr bool FUSED = false, RAW = true;
  static __device__ __forceinline__ void stream(const GemmArgs &ga, const Epi &e, int M, int row_lo, int sk, const Walk &w) {
    if (ga.N % SkinnyW96::BN == 0) gemm_tiles<SkinnyW96, Epi, true>(ga, e, M, row_lo, INT_MAX, sk, w);
    else gemm_tiles<SkinnyN64, Epi, true>(ga, e, M, row_lo, INT_MAX, sk, w);
  }
};

}  // namespace

// raw result part[z][j][n]; returns the numbers of K splits (on the device if the count is there)
Splits gemm_bf16_raw(GemmA A, Rows rows, int K, WSeg seg, float *part, size_t part_elems, int32_t *plan_dev, hipStream_t s) {
  Splits out;
  if (rows.cap <= 0) return out;
  const int N = seg.n_end[2];
  const GemmArgs ga = gemm_args(A, rows, K, seg, nullptr, part);
  const EpiStoreF32 e{part, N};
  const bool w96 = N % SkinnyW96::BN == 0, ring = ring_ok(A, K, seg, N);
  PlanArgs pa = raw_plan_args(N, K, part_elems, ring, cus_of_xcd());
  if (rows.cap <= STREAM_ROWS) {
    out.n = stream_split(pa, rows.cap);
    if (w96) run_tiles<SkinnyW96, true>(ga, e, out.n, s);
    else run_tiles<SkinnyS, true>(ga, e, out.n, s);
    return out;
  }
  GemmPlan pl;
  if (ring) {
    run_planned<RawKind>(ga, e, pa, &pl, plan_dev, s);
    return splits_of(ga, pl, false, plan_dev);
  }
  pa.stream_cols = 0;
  out.n = plan_of(pa, rows.cap, first_on_host(pa, rows.cap)).sk;
  run_tiles<LargeS8, true>(ga, e, out.n, s);
  return out;
}

}  // namespace dy
