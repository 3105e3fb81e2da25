// bf16 q|k|v projection with heads of 128 columns: bias, rotary embedding and the merge into the caches in its epilogue.
#include "gemm_bf16_qkv.h"

namespace dy {

Splits gemm_bf16_qkv128(const GemmArgs &ga, float *part, const QkvOut &out, const PlanArgs &pa, const GemmPlan &pl, int32_t *plan_dev, bool made,
                        hipStream_t s) {
  return run_qkv<128>(ga, part, out, pa, pl, plan_dev, made, s);
}

}  // namespace dy
