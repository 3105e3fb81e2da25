"""Plans made on the host: the choice is that of all candidates priced one by one, whatever the planner leaves out, and costs
a part of that."""
import ctypes as C
import subprocess

import pytest

from paper_2603_08026_amd import build

SOURCE = r"""
#include "%s/gemm_plan.h"
#include <chrono>
#include <random>
using namespace dy::mm;
static GemmPlan every_candidate(const PlanArgs &a, int M) {
  if (M <= STREAM_ROWS && a.stream_cols) return GemmPlan{0, 1, 0, stream_split(a, M), 256};
  GemmPlan p = plan_of(a, M, first_on_host(a, M));
  float first = 2e30f, best = 1e30f;
  for (int h = 0; h < 8; ++h)
    if (first_price(a, p, M, h) < first) { first = first_price(a, p, M, h); p.bm = 32 * (h + 1); }
  GemmPlan q = p;
  for (int shape = 0; shape < 3; ++shape)
    for (int c = 0; c < TILE_CANDIDATES; ++c) {
      const float t = tile_price(a, M, tile_height(a, M, shape, tile_units(c)), tile_split(c));
      if (t < best) { best = t; q = GemmPlan{shape, tile_split(c), M, 1, tile_units(c) * (shape == PLAN_W ? 64 : 32)}; }
    }
  return takes_over(a, M, p, first, q.sk, best) ? q : p;
}
static PlanArgs some(std::mt19937 &r, int *M) {
  const int h = 128 * (1 + r() %% 64), f = 128 * (1 + r() %% 160), q = 128 * (1 + r() %% 100), kind = r() %% 4;
  const long part = (long)exp(std::uniform_real_distribution<double>(12, 20)(r));
  *M = (int)exp(std::uniform_real_distribution<double>(0, 11)(r));
  PlanArgs a = kind == 0 ? raw_plan_args(q, h, part, r() %% 8, 32) : kind == 1 ? swiglu_plan_args(f, h, 32) : down_plan_args(h, f, part, r() %% 8, 32);
  if (kind == 2) a.sum_us = 4.0f;
  if (kind == 3) a.split_ok = a.stream_cols = 0;
  return a;
}
extern "C" int differ(int n) {
  std::mt19937 r(1);
  int bad = 0;
  for (int i = 0; i < n; ++i) {
    int M;
    const PlanArgs a = some(r, &M);
    const GemmPlan p = plan_on_host(a, M), q = every_candidate(a, M);
    bad += p.xl != q.xl || p.sk != q.sk || p.row_hi != q.row_hi || p.sk_tail != q.sk_tail || p.bm != q.bm;
  }
  return bad;
}
extern "C" double cost(int kind, int M) {  // of a plan, against pricing every candidate: the best of several timings of each
  const PlanArgs a = kind == 0 ? raw_plan_args(12288, 4096, 1 << 27, true, 32) : kind == 1 ? swiglu_plan_args(12288, 4096, 32) : down_plan_args(4096, 12288, 1 << 27, true, 32);
  double best[2] = {1e9, 1e9};
  volatile int sink = 0;
  for (int rep = 0; rep < 30; ++rep)
    for (int which = 0; which < 2; ++which) {
      const auto t0 = std::chrono::steady_clock::now();
      for (int i = 0; i < 300; ++i) {
        PlanArgs b = a;
        asm volatile("" : "+m"(b));
        sink += which ? plan_on_host(b, M).bm : every_candidate(b, M).bm;
      }
      const double t = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
      if (t < best[which]) best[which] = t;
    }
  return best[1] / best[0];
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("cost")
    src, so = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O3", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = C.CDLL(so)
    out.cost.restype = C.c_double
    return out


def test_the_choice_is_that_of_all_candidates(lib):
    assert lib.differ(20000) == 0


# measured: 0.27 to 0.47 (1 with every candidate priced)
@pytest.mark.parametrize("rows", [130, 256, 1024, 4096, 20480])
def test_a_plan_costs_a_part_of_pricing_all(lib, rows):
    assert lib.cost(0, rows) < 0.75
