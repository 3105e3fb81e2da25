// bf16 GEMMs with an fp32 result for a row kernel: q|k|v and the out-projection.
#include "gemm_bf16_launch.h"

namespace dy {

// q|k|v (gemm_bf16_qkv.hip, gemm_bf16_qkv64.hip: heads of 128 and 64 columns), or with an empty QkvOut any raw result
Splits gemm_bf16_qkv128(const GemmArgs &ga, float *part, const QkvOut &out, const PlanArgs &pa, int32_t *plan_dev, hipStream_t s);
Splits gemm_bf16_qkv64(const GemmArgs &ga, float *part, const QkvOut &out, const PlanArgs &pa, int32_t *plan_dev, hipStream_t s);

// raw result part[z][j][n], or rows finished as `qkv` says; returns the numbers of K splits (on the device if the count is there)
Splits gemm_bf16_raw(GemmA A, Rows rows, int K, WSeg seg, float *part, size_t part_elems, int32_t *plan_dev, const QkvOut *qkv,
                     hipStream_t s) {
  Splits out;
  if (rows.cap <= 0) return out;
  const int N = seg.n_end[2];
  const GemmArgs ga = gemm_args(A, rows, K, seg, nullptr, part);
  const bool ring = ring_ok(A, K, seg, N);
  // A list with room for most of the tokens is a carried one that holds a few percent of them: K of its GEMMs is split, and they
  // keep to the raw result in a kernel that knows nothing else (8 x 1024 tokens with 330 listed rows, two layers, four
  // steps: 2075 us; in the kernel that can finish rows, which is three times as long, 2091).  All other raw results
  // of planned GEMMs share that one, of which the instruction caches then still hold a part from GEMM to GEMM (five sparse
  // steps of 410 to 5160 rows 0.1 to 1.7 % faster than with the out-projection in a kernel of its own).
  const bool few = rows.count && (size_t)rows.cap * 2 > (qkv ? qkv->tokens : A.a_rows);
  // (Lists whose K is split even when they are full, and a few known rows whose K is, such as a response window's, are in the same
  // place: in the long kernel 307 listed rows of hidden 4096 lost 1.7 %, 360 of 28 over 4 heads 1.9 % of a step.)
  constexpr int FEW_ROWS = 512;
  // (positions come from a division by at least two, rotary table entries from 32-bit offsets)
  if (qkv && (qkv->L < 2 || (size_t)qkv->L * qkv->dh * 4 >= ((size_t)1 << 31))) qkv = nullptr;
  const auto qkv_gemm = qkv && qkv->dh == 64 ? gemm_bf16_qkv64 : gemm_bf16_qkv128;
  PlanArgs pa = raw_plan_args(N, K, part_elems, ring, cus_of_xcd());
  if (rows.cap <= STREAM_ROWS) {
    const EpiStoreF32 e{part, N};
    out.n = stream_split(pa, rows.cap);
    if (N % SkinnyW96::BN == 0) run_tiles<SkinnyW96, true>(ga, e, out.n, s);
    else run_tiles<SkinnyS, true>(ga, e, out.n, s);
    return out;
  }
  if (ring) {
    const GemmPlan pl = plan_here(ga, pa);
    const bool split = plan_known(rows) ? pl.sk > 1 && rows.cap <= FEW_ROWS : !few && plan_on_host(pa, rows.cap).sk > 1;
    if (few || split) {
      run_planned<RawKind<EpiStoreF32>>(ga, EpiStoreF32{part, N}, pa, pl, plan_dev, s);
      return splits_of(ga, pl, false, plan_dev);
    }
    return qkv ? qkv_gemm(ga, part, *qkv, pa, plan_dev, s) : gemm_bf16_qkv128(ga, part, QkvOut{}, pa, plan_dev, s);
  }
  pa.stream_cols = 0;
  out.n = plan_of(pa, rows.cap, first_on_host(pa, rows.cap)).sk;
  run_tiles<LargeS8, true>(ga, EpiStoreF32{part, N}, out.n, s);
  return out;
}

}  // namespace dy
