"""Row tiles of every height and the 192-column tiles of the planned GEMMs: the plans (gemm_plan.h, compiled for the
host), and the layer against the oracle at row counts where each of them runs, with a last tile that is lower than the
others and one that ends inside a block of 16 rows."""
import ctypes as C
import subprocess

import pytest

from paper_2603_08026_amd import build
from synth import workload as W

SMALL = W.LayerShape(hidden=1024, n_heads=8, n_kv_heads=8, head_dim=128, ffn=1536, dtype="bf16")
WIDE = W.LayerShape(hidden=4096, n_heads=32, n_kv_heads=32, head_dim=128, ffn=12288, dtype="bf16")
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
]

SOURCE = r"""
#include "%s/gemm_plan.h"
using namespace dy::mm;
extern "C" void plan(int kind, int N, int K, long part_elems, int count, int *out) {
  const PlanArgs a = kind == 0 ? raw_plan_args(N, K, part_elems, true, 32) : kind == 1 ? swiglu_plan_args(N, K, 32)
                                                                                     : down_plan_args(N, K, part_elems, true, 32);
  const GemmPlan p = plan_on_host(a, count);
  out[0] = p.xl == PLAN_X ? 256 : p.xl == PLAN_W ? 192 : 128;
  out[1] = p.sk; out[2] = p.bm;
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
    seen = set()
    for s, count, plans in CASES:
        gemms = {"qkv": (0, s.dq + 2 * s.dkv, s.hidden), "oproj": (0, s.hidden, s.dq), "gate_up": (1, s.ffn, s.hidden),
                 "down": (2, s.hidden, s.ffn)}
        t = _tokens(count)
        part = max(16 * min(t, 2048) * s.dq, t * max(s.dq + 2 * s.dkv, s.hidden))  # the context's fp32 scratch
        for name, want in plans.items():
            kind, n, k = gemms[name]
            out = (C.c_int * 3)()
            lib.plan(kind, n, k, C.c_long(part), count, out)
            assert tuple(out) == want, (count, name, tuple(out))
            seen.add((out[0], out[2]))
    assert {(128, 32 * i) for i in range(1, 9)} <= seen and {c for c, _ in seen} == {128, 192, 256}


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
