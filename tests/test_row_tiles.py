"""Row tiles of every height and the 192-column tiles of the planned GEMMs: the plans (gemm_plan.h, compiled for the
host), and the layer against the oracle at row counts where each of them runs, with a last tile that is lower than the
others and one that ends inside a block of 16 rows.  Lists are planned on the device (test_gpu_device_plans.py: as the host
does); a dense step of as many rows runs the host's plan itself."""
import ctypes as C
import subprocess

import pytest

from paper_2603_08026_amd import build
from synth import workload as W

SMALL = W.LayerShape(hidden=1024, n_heads=8, n_kv_heads=8, head_dim=128, ffn=1536, dtype="bf16")
WIDE = W.LayerShape(hidden=4096, n_heads=32, n_kv_heads=32, head_dim=128, ffn=12288, dtype="bf16")
FFN = W.LayerShape(hidden=512, n_heads=4, n_kv_heads=4, head_dim=128, ffn=6144, dtype="bf16")
# (layer, rows, {GEMM: (columns, K splits, rows of a tile)})
CASES = [
    (SMALL, 129, {"qkv": (128, 2, 32), "gate_up": (128, 1, 32), "down": (128, 3, 32), "oproj": (128, 2, 32)}),
    (SMALL, 541, {"qkv": (128, 1, 64), "gate_up": (128, 1, 64), "oproj": (128, 2, 64), "down": (128, 3, 64)}),
    (SMALL, 795, {"qkv": (128, 1, 96), "gate_up": (128, 1, 96), "down": (128, 3, 96)}),
    (SMALL, 1165, {"qkv": (128, 1, 128), "gate_up": (128, 1, 128)}),
    (SMALL, 1498, {"qkv": (128, 1, 160), "gate_up": (128, 1, 160)}),
    (SMALL, 1794, {"qkv": (128, 1, 192), "gate_up": (128, 1, 192)}),
    (SMALL, 2127, {"qkv": (128, 1, 224), "gate_up": (128, 1, 224), "oproj": (128, 1, 96), "down": (128, 1, 96)}),
    (SMALL, 2645, {"qkv": (128, 1, 256), "gate_up": (256, 1, 128)}),
    (SMALL, 2867, {"qkv": (256, 1, 160), "gate_up": (192, 1, 192)}),
    (SMALL, 3570, {"qkv": (256, 1, 192), "gate_up": (256, 1, 192)}),
    (SMALL, 4088, {"qkv": (192, 1, 256), "gate_up": (192, 1, 256), "oproj": (128, 1, 128), "down": (128, 1, 128)}),
    (WIDE, 330, {"gate_up": (192, 1, 192), "down": (128, 4, 192)}),
    (WIDE, 511, {"gate_up": (192, 1, 256)}),
    (WIDE, 757, {"gate_up": (192, 1, 192)}),
    (FFN, 387, {"gate_up": (256, 1, 96)}),
    (FFN, 417, {"gate_up": (256, 1, 96)}),
    (FFN, 483, {"gate_up": (192, 1, 128)}),
    (FFN, 1026, {"gate_up": (256, 1, 224)}),
    (FFN, 1122, {"gate_up": (256, 1, 256)}),
    (FFN, 2562, {"down": (128, 5, 224)}),
    (SMALL, 2244, {"gate_up": (128, 1, 256)}),
    (SMALL, 2724, {"qkv": (256, 1, 160), "gate_up": (192, 1, 192)}),
    (SMALL, 4099, {"qkv": (256, 1, 224), "down": (128, 1, 160)}),
    (SMALL, 4899, {"qkv": (256, 1, 256)}),
    (WIDE, 258, {"down": (256, 8, 160)}),
    (WIDE, 579, {"down": (256, 5, 224)}),
    (WIDE, 675, {"qkv": (192, 1, 192), "down": (256, 5, 256)}),
]

SOURCE = r"""
#include "%s/gemm_plan.h"
using namespace dy::mm;
extern "C" void plan(int kind, int N, int K, long part_elems, int count, int *out) {
  const PlanArgs a = kind == 0 ? raw_plan_args(N, K, part_elems, true, 32) : kind == 1 ? swiglu_plan_args(N, K, 32)
                                                                                     : down_plan_args(N, K, part_elems, true, 32);
  const GemmPlan p = plan_on_host(a, count);
  out[0] = p.xl == PLAN_X ? 256 : p.xl == PLAN_W ? 192 : 128;
  out[1] = p.sk; out[2] = p.bm; out[3] = p.row_hi;
  out[4] = past_l2((kind == 1 ? 2 : 1) * N, K);
}
"""


def _tokens(count):
    return max(1, -(-count // 1400)) * 1400


def test_cases_run_the_tiles_they_name(tmp_path):
    src, so = str(tmp_path / "plan.cpp"), str(tmp_path / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = C.CDLL(so)
    seen, blocks = set(), set()
    for s, count, plans in CASES:
        gemms = {"qkv": (0, s.dq + 2 * s.dkv, s.hidden), "oproj": (0, s.hidden, s.dq), "gate_up": (1, s.ffn, s.hidden),
                 "down": (2, s.hidden, s.ffn)}
        t = _tokens(count)
        part = max(16 * min(t, 2048) * s.dq, t * max(s.dq + 2 * s.dkv, s.hidden))  # the context's fp32 scratch
        for name, want in plans.items():
            kind, n, k = gemms[name]
            out = (C.c_int * 5)()
            lib.plan(kind, n, k, C.c_long(part), count, out)
            assert tuple(out[:3]) == want, (count, name, tuple(out))
            seen.add((out[0], out[2]))
        for name, (kind, n, k) in gemms.items():  # 16-row blocks of a wave in the whole tiles and in the last one
            out = (C.c_int * 5)()
            lib.plan(kind, n, k, C.c_long(part), count, out)
            if out[3] == count:
                unit = 64 if out[0] == 192 else 32
                form = {0: "raw", 1: "swiglu", 2: "down" if out[1] == 1 else "raw sums"}[kind]
                blocks |= {(form, out[0], -(-r // unit)) for r in (min(out[2], count), count % out[2]) if r}
    assert {(128, 32 * i) for i in range(1, 9)} <= seen and {c for c, _ in seen} == {128, 192, 256}
    # every form of result, column width and number of blocks that plans of these layers come to (192 columns: heights of 64 rows)
    for form, cols, heights in (("raw", 128, range(1, 9)), ("raw", 192, range(2, 5)), ("raw", 256, range(1, 9)),
                                ("swiglu", 128, range(1, 9)), ("swiglu", 192, range(1, 5)), ("swiglu", 256, range(1, 9)),
                                ("raw sums", 128, range(1, 9)), ("raw sums", 256, range(4, 9)), ("down", 128, range(1, 6))):
        assert {(form, cols, h) for h in heights} <= blocks, (form, cols, sorted(blocks))


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES)))
def test_layer_in_tiles_of_this_height(case):
    from paper_2603_08026_amd.layer import Layer
    from tests.helpers import rand_weights
    from tests.test_gpu_planned_gemm import _check
    shape, count, _ = CASES[case]
    print("row tiles", case, count, flush=True)
    B = _tokens(count) // 1400
    lay = Layer.from_shape(shape, B, 1400)
    w = rand_weights(shape, 57, bias=True)
    lay.set_weights(w)
    _check(lay, w, shape, B, 1400, count, count)
    lay.close()


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES)))
def test_dense_step_of_as_many_rows(case):
    """The host's plans: keys, values and output rows of a dense step against those of the list of all its tokens."""
    import torch
    from paper_2603_08026_amd import binding as Bd
    from paper_2603_08026_amd.layer import Layer
    from tests.helpers import TOL, rand_weights
    shape, count, _ = CASES[case]
    print("dense rows", case, count, flush=True)
    lay = Layer.from_shape(shape, 1, count)
    lay.set_weights(rand_weights(shape, 58, bias=True))
    x = torch.randn(1, count, shape.hidden, generator=torch.Generator().manual_seed(59)).to(torch.bfloat16).cuda()
    lay.full_step(x)
    dense = [t.float().clone() for t in (lay.k, lay.v, lay.out)]
    every = Bd.IndexList(torch.arange(count, dtype=torch.int32, device="cuda"), torch.tensor([0, count], dtype=torch.int32, device="cuda"))
    for t in (lay.k, lay.v, lay.out):
        t.fill_(float("nan"))
    q = torch.zeros(count, shape.dq, dtype=torch.bfloat16, device="cuda")
    lay.ctx.qkv_refresh(lay.w, x, every, 1, count, lay.cache, q)
    lay.ctx.salient_ffn(lay.w, x, lay.c, every, 1, count, lay.out)
    for name, a, b in zip(("k", "v", "out"), dense, (lay.k, lay.v, lay.out)):
        err = float((a - b.float()).abs().max() / a.abs().max())
        assert err <= TOL["bf16"], (name, err)
    lay.close()


# Rows that all lie in one row tile of more than half the height: weights copied past the L2, in loops that exist for some of the
# tiles' shapes only.
# (matrices of 16 MiB and more; the same loops copy those of "small" through the L2)
ONE_TILE = {"wide": (WIDE, [143, 161, 224, 245]), "grouped": (W.DREAM, [129, 192, 200, 256])}
SMALL_TILE = {"small": (SMALL, [129, 161, 224, 256])}


def _one_tile_plans(lib, s, count):
    """{GEMM: (columns, K splits, rows of a tile)} of the GEMMs that have `count` rows in one such tile"""
    part = 16 * 2048 * s.dq
    plans = {}
    for name, (kind, n, k) in {"qkv": (0, s.dq + 2 * s.dkv, s.hidden), "oproj": (0, s.hidden, s.dq), "gate_up": (1, s.ffn, s.hidden),
                               "down": (2, s.hidden, s.ffn)}.items():
        out = (C.c_int * 5)()
        lib.plan(kind, n, k, C.c_long(part), count, out)
        if out[4] and count <= out[2] and -(-count // (64 if out[0] == 192 else 32)) > (2 if out[0] == 192 else 4):
            plans[name] = tuple(out[:3])
    return plans


def test_few_rows_take_the_shapes_that_have_loops_for_them(tmp_path):
    src, so = str(tmp_path / "plan.cpp"), str(tmp_path / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = C.CDLL(so)
    for dims in ((4096, 32, 32, 12288), (3584, 28, 4, 18944), (512, 4, 1, 1536), (1024, 8, 8, 3072), (2048, 16, 4, 5632),
                 (5120, 40, 8, 25600), (8192, 64, 8, 28672), (4096, 32, 8, 14336)):
        s = W.LayerShape(hidden=dims[0], n_heads=dims[1], n_kv_heads=dims[2], head_dim=128, ffn=dims[3], dtype="bf16")
        for count in range(1, 513):
            for name, (cols, splits, _) in _one_tile_plans(lib, s, count).items():
                assert cols == 128 and (splits > 1 or name != "down") or (cols, name) == (256, "gate_up"), (dims, count, name)
    # the counts of the test below run every such loop
    seen = {(name, p[0], p[2]) for s, counts in ONE_TILE.values() for n in counts for name, p in _one_tile_plans(lib, s, n).items()}
    assert {(name, cols, h) for name, cols in (("qkv", 128), ("gate_up", 128), ("gate_up", 256), ("down", 128)) for h in (160, 192, 224, 256)} <= seen


@pytest.mark.gpu
@pytest.mark.parametrize("case", sorted(ONE_TILE) + sorted(SMALL_TILE))
def test_layer_of_rows_in_one_tile(case):
    from paper_2603_08026_amd.layer import Layer
    from tests.helpers import rand_weights
    from tests.test_gpu_planned_gemm import _check
    shape, counts = {**ONE_TILE, **SMALL_TILE}[case]
    lay = Layer.from_shape(shape, 1, 600)
    w = rand_weights(shape, 60, bias=True)
    lay.set_weights(w)
    for count in counts:
        for cap in (count, 600) if count == counts[0] else (count,):
            print("rows in one tile", case, count, cap, flush=True)
            _check(lay, w, shape, 1, 600, count, cap)
    lay.close()
