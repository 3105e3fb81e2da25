"""The bf16 GEMMs' launch rules (gemm_plan.h), compiled for the host: no GPU needed.  What the GPU tests of the
planned GEMMs say that their cases run is checked here against the rules, so that a change of the prices cannot
quietly empty those cases."""
import ctypes as C
import subprocess

import pytest

from paper_2603_08026_amd import build
from synth import workload as W
from tests.test_gpu_planned_gemm import HALF, NO_SUMS_CAP, REGIMES, SHAPE

SOURCE = r"""
#include "%s/gemm_plan.h"
using namespace dy::mm;
extern "C" int groups_ok(int end0, int end1) { return ring_groups_ok(end0, end1); }
// 0: nothing, 1: weight-streaming tiles, 2: row tiles, 3: eight-wave shapes; for a GEMM whose kernel cannot make its plan
extern "C" int way(int cap, int streams, int ring, int listed, int made) { return (int)way_with(way_of(cap, streams, ring), listed, cap, made); }
extern "C" int ahead(int cap, int streams, int ring, int listed) { return wants_plan(way_of(cap, streams, ring), listed, cap); }
// raw result of `cap` rows (listed: of a list, whose count is on the device) of `tokens`: in the kernel that can finish rows?
extern "C" int finishes(int N, int K, long part_elems, int listed, int cap, long tokens) {
  const bool few = few_of_room(listed, cap, tokens) || few_results(plan_known(listed, cap), cap, N);
  return finishing_kernel(few, plan_on_host(raw_plan_args(N, K, part_elems, true, 32), cap));
}
// kind 0: raw result, 1: gate|up, 2: down; the plan of a list with `count` of `cap` entries (cap < 0: count known on
// the host) -> columns of the row tiles (0: weight-streaming tiles alone), splits, rows in row tiles, splits behind them,
// planned on the device, sum kernel
extern "C" void plan(int kind, int N, int K, long part_elems, int count, int cap, int *out) {
  PlanArgs a = kind == 0 ? raw_plan_args(N, K, part_elems, true, 32) : kind == 1 ? swiglu_plan_args(N, K, 32)
                                                                                : down_plan_args(N, K, part_elems, true, 32);
  const bool known = plan_known(cap >= 0, cap < 0 ? count : cap);
  const int c = cap < 0 ? count : cap;
  out[5] = kind == 0 ? 1 : kind == 2 ? down_has_sums(a, c, known) : 0;
  if (kind == 2 && !out[5]) a.split_ok = a.stream_cols = 0;
  const GemmPlan p = plan_on_host(a, known ? c : count);
  out[0] = p.row_hi == 0 ? 0 : p.xl ? 256 : 128;
  out[1] = p.sk; out[2] = p.row_hi; out[3] = p.sk_tail; out[4] = !known;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return C.CDLL(so)


class Plan:
    def __init__(self, lib, shape, gemm, count, cap, tokens):
        d, dq, dkv, f = shape.hidden, shape.dq, shape.dkv, shape.ffn
        kind, n, k = {"qkv": (0, dq + 2 * dkv, d), "oproj": (0, d, dq), "gate_up": (1, f, d), "down": (2, d, f)}[gemm]
        part = max(16 * min(tokens, 2048) * dq, tokens * max(dq + 2 * dkv, d))  # the context's fp32 scratch
        out = (C.c_int * 6)()
        lib.plan(kind, n, k, C.c_long(part), count, cap, out)
        self.cols, self.splits, self.tiled_rows, self.tail_splits, self.on_device, self.sums = out
        self.streams_tail = 0 < self.tiled_rows < count


@pytest.mark.parametrize("end", [8, 16, 24, 40, 4096 + 8, 4096 + 16])
def test_matrix_ends_inside_a_group_of_permuted_rows_are_not_for_the_ring_loop(lib, end):
    assert not lib.groups_ok(end, 8192)
    assert not lib.groups_ok(4096, end)


@pytest.mark.parametrize("dq,dkv", [(4096, 4096), (3584, 512), (256, 64), (128, 128)])
def test_ends_of_the_stacked_projections_are(lib, dq, dkv):
    assert lib.groups_ok(dq, dq + dkv)
    assert lib.groups_ok(dkv, 2 * dkv)


def test_row_tiles_of_counted_rows_have_a_plan(lib):
    for cap in (0, 1, 128, 129, 256, 257, 5000):
        for streams in (0, 1):
            for ring in (0, 1):
                for listed in (0, 1):
                    base = 0 if cap == 0 else 1 if streams and cap <= 128 else 2 if ring else 3
                    device = base == 2 and listed and cap > 256  # its plan is made on the device
                    assert lib.ahead(cap, streams, ring, listed) == int(device)
                    assert lib.way(cap, streams, ring, listed, 1) == base
                    assert lib.way(cap, streams, ring, listed, 0) == (3 if device else base)


@pytest.mark.parametrize("case", range(len(REGIMES)))
def test_cases_of_the_gpu_test_run_the_plans_they_name(lib, case):
    shape, count, cap, plans = REGIMES[case]
    tokens = 4200 if cap > 2200 else 2200
    for gemm, want in plans.items():
        p = Plan(lib, shape, gemm, count, cap, tokens)
        assert p.on_device and (gemm != "down" or p.sums)
        assert (p.cols, p.splits, p.tiled_rows, p.tail_splits) == want, gemm


@pytest.mark.parametrize("count", [1, 128, 129, 330, 640])
def test_capacities_around_the_range_without_a_sum_kernel(lib, count):
    for cap, sums in ((1000, True), (NO_SUMS_CAP, False), (4200, True)):
        p = Plan(lib, SHAPE, "down", count, cap, 4200)
        assert p.on_device and bool(p.sums) == sums
        if not sums:
            assert p.splits == 1 and p.tiled_rows == count  # no split and no streamed rows, however few they are
        elif count <= 128:
            assert p.tiled_rows == 0 and p.tail_splits > 1  # weight-streaming tiles alone
        else:
            assert p.splits == 3


# rows, capacity, FFN width of test_gpu_kernels.py's test of a short last row tile (4096 hidden, 32 over 16 heads) ->
# the GEMMs that hand the rows behind the full tiles to the weight-streaming tiles, with how many splits
@pytest.mark.parametrize("count,cap,ffn,streamed", [
    (2075, 2075, 4096, {"qkv": 2, "oproj": 4, "gate_up": 1}), (2060, 2075, 4096, {"qkv": 2, "oproj": 4, "gate_up": 1}),
    (1990, 2075, 4096, {}), (1819, 1819, 12288, {}), (1800, 1819, 12288, {})])
def test_streamed_rows_of_a_short_last_row_tile(lib, count, cap, ffn, streamed):
    shape = W.LayerShape(hidden=4096, n_heads=32, n_kv_heads=16, head_dim=128, ffn=ffn, dtype="bf16")
    for gemm in ("qkv", "oproj", "gate_up", "down"):
        p = Plan(lib, shape, gemm, count, cap, 2200)
        assert p.streams_tail == (gemm in streamed), gemm
        assert not p.streams_tail or p.tail_splits == streamed[gemm], gemm


@pytest.mark.parametrize("count,cap,cols,streams", [(32668, 32768, 128, False), (16411, 16411, 256, True),
                                                    (16400, 16411, 256, True), (9000, 16411, 256, False)])
def test_plans_of_the_many_row_cases(lib, count, cap, cols, streams):
    shape = W.LayerShape(hidden=1024, n_heads=4, n_kv_heads=2, head_dim=128, ffn=512, dtype="bf16")
    p = Plan(lib, shape, "qkv", count, cap, 32768 if cap > 17600 else 17600)
    assert p.streams_tail == streams and p.splits == 1 and p.tail_splits == 1
    assert p.cols == cols


# (hidden, query heads, KV heads, FFN width), GEMM, rows -> columns and K splits of the faster of the two sets' choices, both of
# which were timed with the sums of their splits
@pytest.mark.parametrize("dims,gemm,count,cols,splits", [
    ((4096, 32, 32, 12288), "qkv", 256, 128, 2), ((4096, 32, 32, 12288), "oproj", 960, 128, 2),
    ((4096, 32, 32, 12288), "oproj", 1024, 128, 2), ((4096, 32, 32, 12288), "oproj", 1500, 256, 2),
    ((3584, 28, 4, 18944), "oproj", 1000, 128, 2), ((3584, 28, 4, 18944), "qkv", 768, 128, 2),
    ((4096, 32, 32, 12288), "qkv", 400, 128, 1), ((4096, 32, 32, 12288), "qkv", 512, 128, 1),
    ((3584, 28, 4, 18944), "qkv", 1200, 128, 1), ((4096, 32, 32, 12288), "oproj", 1100, 128, 1), ((2048, 16, 16, 5632), "oproj", 640, 128, 2),
    ((1024, 8, 8, 2816), "qkv", 512, 128, 1), ((1024, 8, 8, 2816), "oproj", 1700, 128, 1),
    ((4096, 32, 32, 12288), "oproj", 2000, 128, 1), ((5120, 40, 8, 13824), "oproj", 3670, 256, 1),
    ((6144, 48, 8, 16384), "oproj", 3310, 256, 1), ((6144, 48, 8, 16384), "oproj", 4030, 256, 1)])
def test_plans_of_timed_pairs(lib, dims, gemm, count, cols, splits):
    d, h, kv, f = dims
    p = Plan(lib, W.LayerShape(hidden=d, n_heads=h, n_kv_heads=kv, head_dim=128, ffn=f, dtype="bf16"), gemm, count, 6144, 6144)
    assert (p.cols, p.splits, p.tiled_rows) == (cols, splits, count)


# layer (hidden, query heads, KV heads), rows (capacity of the list), tokens, list -> q|k|v in the kernel that can finish rows
@pytest.mark.parametrize("dims,cap,tokens,listed,finishes", [
    ((4096, 32, 32), 20480, 20480, False, True), ((4096, 32, 32), 1100, 1100, False, True),
    ((4096, 32, 32), 200, 200, False, False),                                     # known rows whose K is split
    ((3584, 28, 4), 560, 560, False, False), ((3584, 28, 4), 1600, 1600, False, True),
    ((4096, 32, 0), 768, 3072, False, False), ((4096, 32, 0), 1024, 4096, False, False),  # q of response windows
    ((4096, 32, 32), 2064, 20480, True, True), ((4096, 32, 32), 5160, 20480, True, True),
    ((4096, 32, 32), 2064, 4128, True, True), ((4096, 32, 32), 2064, 4127, True, False),  # room for more than half of the tokens
    ((4096, 32, 32), 8192, 8192, True, False),
    ((3584, 28, 4), 360, 3600, True, False),                                      # lists whose K is split when they are full
    ((512, 4, 4), 256, 16384, True, True), ((512, 4, 4), 257, 16384, True, False),  # few results of a plan on the device
    ((1024, 8, 8), 1099, 16384, True, False), ((1024, 8, 8), 1100, 16384, True, True), ((1024, 8, 8), 400, 400, False, True),
    ((2048, 16, 15), 1099, 16384, True, False), ((2048, 16, 16), 1099, 16384, True, True), ((2048, 16, 16), 310, 16384, True, True)])
def test_kernel_of_the_projections(lib, dims, cap, tokens, listed, finishes):
    d, h, kv = dims
    part = C.c_long(max(16 * min(tokens, 2048) * h * 128, tokens * max(128 * (h + 2 * kv), d)))
    assert lib.finishes(128 * (h + 2 * kv), d, part, int(listed), cap, C.c_long(tokens)) == int(finishes)


def test_regimes_of_lists_of_half_the_tokens(lib):
    """Each of them is in the kernel that finishes rows, among them one whose streamed rows the row kernel finishes."""
    streamed = 0
    for case in HALF:
        shape, count, cap, plans = REGIMES[case]
        tokens = 4 * ((cap + 1) // 2)
        part = C.c_long(max(16 * min(tokens, 2048) * shape.dq, tokens * max(shape.dq + 2 * shape.dkv, shape.hidden)))
        assert lib.finishes(shape.dq + 2 * shape.dkv, shape.hidden, part, 1, cap, C.c_long(tokens)) == 1, case
        for gemm, want in plans.items():
            p = Plan(lib, shape, gemm, count, cap, tokens)
            assert (p.cols, p.splits, p.tiled_rows, p.tail_splits) == want, (case, gemm)
            streamed += gemm == "qkv" and p.splits == 1 and p.streams_tail
    assert HALF and streamed
