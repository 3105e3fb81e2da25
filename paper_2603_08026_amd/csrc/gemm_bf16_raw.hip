// bf16 GEMMs with an fp32 result for a row kernel: q|k|v and the out-projection.
#include "gemm_bf16_launch.h"

namespace dy {

// q|k|v of a dense step of many rows, the values straight into their cache (gemm_bf16_qkv.hip)
Splits gemm_bf16_qkv(const GemmArgs &ga, float *part, const DirectCols &direct, const PlanArgs &pa, hipStream_t s);

// raw result part[z][j][n]; returns the numbers of K splits (on the device if the count is there)
Splits gemm_bf16_raw(GemmA A, Rows rows, int K, WSeg seg, float *part, size_t part_elems, int32_t *plan_dev, DirectCols direct,
                     hipStream_t s) {
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
  if (ring) {
    // Dense steps from DIRECT_ROWS rows on: 20480 rows of 12288 columns, GEMM and row kernel together 1835 -> 1735 us.  The line
    // is the smallest measured count from which no layer loses (dense steps without / with, us: hidden 4096, 2048 rows 756 /
    // 751, 4096 rows 1410 / 1390, 8192 rows 2780 / 2741; hidden 3584 with four KV heads 799 / 801, 1511 / 1501, 2932 / 2937;
    // hidden 2048 258 / 254, 453 / 448, 837 / 808; hidden 1024 115 / 116, 183 / 180, 336 / 327, and 82 / 85 at 1024 rows).  Lists
    // stay with the raw result: the kernel is another one than the out-projection's, whose instructions the caches
    // still hold from layer to layer, and few rows lose more by that than they gain (loop of 8 x 1024 tokens with 330 listed
    // rows 2119 -> 2149 us a pass, 410 rows of a list 302 -> 306 us a step; 2064 rows 812 -> 808, 5160 rows 1872 -> 1859,
    // but how many of a list exist is known to the device alone).
    if (direct.out && !rows.idx && !rows.count && rows.cap >= DIRECT_ROWS) return gemm_bf16_qkv(ga, part, direct, pa, s);
    const GemmPlan pl = plan_here(ga, pa);
    run_planned<RawKind<EpiStoreF32>>(ga, e, pa, pl, plan_dev, s);
    return splits_of(ga, pl, false, plan_dev);
  }
  pa.stream_cols = 0;
  out.n = plan_of(pa, rows.cap, first_on_host(pa, rows.cap)).sk;
  run_tiles<LargeS8, true>(ga, e, out.n, s);
  return out;
}

}  // namespace dy
