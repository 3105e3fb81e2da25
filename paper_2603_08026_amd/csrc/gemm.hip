// Dispatch of the salient-row GEMMs by storage type: gemm_f32.hip, gemm_bf16_*.hip.
#include "kernels.h"

namespace dy {

void gemm_f32_raw(GemmA, Rows, int, WSeg, float *, hipStream_t);
void gemm_f32_down(GemmA, Rows, int, int, const void *, const float *, void *, hipStream_t);

PlanJob gemm_bf16_raw_plan(GemmA, Rows, int, WSeg, size_t, int32_t *, const QkvOut &);
PlanJob gemm_bf16_swiglu_plan(Rows, int, int, int32_t *);
PlanJob gemm_bf16_down_plan(Rows, int, int, size_t, int32_t *);
Splits gemm_bf16_raw(GemmA, Rows, int, WSeg, float *, size_t, int32_t *, const PlanJob &, const QkvOut &, hipStream_t);
void gemm_bf16_swiglu(GemmA, Rows, int, int, const void *, const void *, void *, const PlanJob &, hipStream_t);
void gemm_bf16_down(GemmA, Rows, int, int, const void *, const float *, void *, float *, size_t, const PlanJob &, hipStream_t);

PlanJob plan_gemm_raw(DType t, GemmA A, Rows rows, int K, WSeg seg, size_t part_elems, int32_t *plan, const QkvOut &qkv) {
  return t == F32 ? PlanJob{} : gemm_bf16_raw_plan(A, rows, K, seg, part_elems, plan, qkv);
}
PlanJob plan_gemm_swiglu(Rows rows, int K, int N, int32_t *plan) { return gemm_bf16_swiglu_plan(rows, K, N, plan); }
PlanJob plan_gemm_down(DType t, Rows rows, int K, int N, size_t scratch_elems, int32_t *plan) {
  return t == F32 ? PlanJob{} : gemm_bf16_down_plan(rows, K, N, scratch_elems, plan);
}

Splits launch_gemm_raw(DType t, GemmA A, Rows rows, int K, WSeg seg, float *part, size_t part_elems,
                       int32_t *plan, const PlanJob &job, const QkvOut &qkv, hipStream_t s) {
  if (t == F32) {
    gemm_f32_raw(A, rows, K, seg, part, s);
    return Splits{};
  }
  return gemm_bf16_raw(A, rows, K, seg, part, part_elems, plan, job, qkv, s);
}

void launch_gemm_swiglu(const void *a, Rows rows, int K, int N, const void *w_gate,
                        const void *w_up, void *act, const PlanJob &job, hipStream_t s) {
  gemm_bf16_swiglu(GemmA{a, nullptr, K}, rows, K, N, w_gate, w_up, act, job, s);
}

void launch_gemm_down(DType t, const void *a, Rows rows, int K, int N, const void *w_down, const float *h,
                      void *out_cache, float *scratch, size_t scratch_elems, const PlanJob &job, hipStream_t s) {
  const GemmA A{a, nullptr, K};
  if (t == F32) gemm_f32_down(A, rows, K, N, w_down, h, out_cache, s);
  else gemm_bf16_down(A, rows, K, N, w_down, h, out_cache, scratch, scratch_elems, job, s);
}

}  // namespace dy
