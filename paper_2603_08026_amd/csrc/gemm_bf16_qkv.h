// q|k|v projections whose rows the GEMM finishes where K is not split (a source file per head size: each holds the paths of
// its tiles for every height).
#pragma once
#include "gemm_bf16_launch.h"

namespace dy {

namespace {

// r / d = (r * mul) >> (32 + shift) for every r below 2^31 (d >= 2): 2^(32 + shift) exceeds 2^31 times mul's excess over the
// exact quotient's, which is below d
inline void division_by(uint32_t d, uint32_t *mul, uint32_t *shift) {
  uint32_t s = 0;
  while (((uint64_t)2 << s) < d) ++s;
  *shift = s;
  *mul = (uint32_t)(((uint64_t)1 << (32 + s)) / d + 1);
}

template <int DH>
Splits run_qkv(const GemmArgs &ga, float *part, const QkvOut &out, const PlanArgs &pa, const GemmPlan &pl, int32_t *plan_dev, bool made,
               hipStream_t s) {
  EpiQkv<DH> e;
  e.out = part;
  e.ldo = ga.N;
  e.o = out;
  e.l_mul = e.l_shift = 0;
  if (out.tab) division_by((uint32_t)out.L, &e.l_mul, &e.l_shift);
  with_once(past_l2(ga.N, ga.K), [&](auto once) { run_planned<RawKind<EpiQkv<DH>, decltype(once)::value>>(ga, e, pa, pl, plan_dev, made, s); });
  return splits_of(ga, pl, out.tab != nullptr, plan_dev);
}

}  // namespace

}  // namespace dy
