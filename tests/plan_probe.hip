// The plans that the planned GEMMs make on the device (plan_on_device), beside those of the host planner, for the tests.
#include <vector>
#include "../paper_2603_08026_amd/csrc/gemm_plan.h"

using namespace dy::mm;

namespace {

__global__ __launch_bounds__(256) void k_plans(PlanArgs a, const int *rows, GemmPlan *out) {
  __shared__ uint32_t words[8];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const GemmPlan p = plan_on_device(a, rows[blockIdx.x], wave, words);
  if (threadIdx.x == 0) out[blockIdx.x] = p;
}

bool same(const GemmPlan &p, const GemmPlan &q) {
  return p.xl == q.xl && p.sk == q.sk && p.row_hi == q.row_hi && p.sk_tail == q.sk_tail && p.bm == q.bm;
}

// Whether plan d is a choice that prices known to within a share e allow.  The device keeps 17 bits of a price and rounds
// its products otherwise (fused multiply-adds).
bool allowed(const PlanArgs &a, int M, const GemmPlan &d, float e) {
  if (M <= STREAM_ROWS && a.stream_cols) return same(d, plan_on_host(a, M));
  float least = 1e30f, best = 1e30f;
  for (int c = 0; c < PLAN_CANDIDATES; ++c) least = fminf(least, plan_price(a, M, c));
  for (int shape = 0; shape < 3; ++shape)
    for (int c = 0; c < TILE_CANDIDATES; ++c)
      best = fminf(best, tile_price(a, M, tile_height(a, M, shape, tile_units(c)), tile_split(c)));
  for (int c = 0; c < PLAN_CANDIDATES; ++c) {
    if (plan_price(a, M, c) > (1 + e) * least) continue;
    GemmPlan p = plan_of(a, M, c);
    float first = 2e30f;
    for (int h = 0; h < 8; ++h) first = fminf(first, first_price(a, p, M, h));
    for (int shape = 0; shape < 3; ++shape)
      for (int k = 0; k < TILE_CANDIDATES; ++k) {
        const int sk = tile_split(k), unit = shape == PLAN_W ? 64 : 32;
        if (tile_price(a, M, tile_height(a, M, shape, tile_units(k)), sk) > (1 + e) * best) continue;
        const bool up = takes_over(a, M, p, first, sk, best * (1 - e)), down = takes_over(a, M, p, first, sk, best * (1 + e));
        if (up && same(d, GemmPlan{shape, sk, M, 1, tile_units(k) * unit})) return true;
        if (down) continue;
        for (int h = 0; h < 8; ++h) {
          p.bm = 32 * (h + 1);
          if (first_price(a, p, M, h) <= (1 + e) * first && same(d, p)) return true;
        }
      }
  }
  return false;
}

}  // namespace

// kind 0: raw result, 1: gate|up, 2: down; plans of n row counts.  out[0]: plans that are not the host's, out[1]: those among
// them that no rounding of the prices explains, out[2], out[3], out[4]: the device's plans with 128, 256, 192 columns,
// out[5]: a row count of out[1].  Returns 0, or the HIP error.
extern "C" int compare_plans(int kind, int N, int K, long part_elems, int n, const int *rows, int *out) {
  const PlanArgs a = kind == 0 ? raw_plan_args(N, K, part_elems, true, 32) : kind == 1 ? swiglu_plan_args(N, K, 32) : down_plan_args(N, K, part_elems, true, 32);
  int *d_rows = nullptr;
  GemmPlan *d_out = nullptr;
  std::vector<GemmPlan> got(n);
  hipError_t e = hipMalloc(&d_rows, n * sizeof(int));
  if (e == hipSuccess) e = hipMalloc(&d_out, n * sizeof(GemmPlan));
  if (e == hipSuccess) e = hipMemcpy(d_rows, rows, n * sizeof(int), hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    k_plans<<<n, 256>>>(a, d_rows, d_out);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpy(got.data(), d_out, n * sizeof(GemmPlan), hipMemcpyDeviceToHost);
  (void)hipFree(d_rows);
  (void)hipFree(d_out);
  if (e != hipSuccess) return (int)e;
  for (int i = 0; i < 6; ++i) out[i] = 0;
  for (int i = 0; i < n; ++i) {
    ++out[2 + got[i].xl];
    if (same(got[i], plan_on_host(a, rows[i]))) continue;
    ++out[0];
    if (allowed(a, rows[i], got[i], 5e-5f)) continue;
    ++out[1];
    out[5] = rows[i];
  }
  return 0;
}
