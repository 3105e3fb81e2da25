// bf16 q|k|v projection of many rows whose value columns go straight into the value cache.
#include "gemm_bf16_launch.h"

namespace dy {

Splits gemm_bf16_qkv(const GemmArgs &ga, float *part, const DirectCols &direct, const PlanArgs &pa, hipStream_t s) {
  EpiStoreDirect e;
  e.out = part;
  e.ldo = ga.N;
  e.direct = direct;
  const GemmPlan pl = plan_here(ga, pa);
  if (pl.sk > 1) e.direct.lo = INT_MAX;  // sums of a split are finished by the row kernel
  run_planned<RawKind<EpiStoreDirect>>(ga, e, pa, pl, nullptr, s);
  return splits_of(ga, pl, true, nullptr);
}

}  // namespace dy
