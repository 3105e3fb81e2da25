"""The two forms of the approximate update at head_dim 128 (compact_form in kernels.h): the rule, compiled for the host,
and steps whose sequences stand on both sides of it, against the oracle, twice in a row with other candidates, so
that a value residual that a step left behind shows in the next."""
import ctypes as C
import subprocess

import numpy as np
import pytest

from oracle import dyllm_oracle as O
from paper_2603_08026_amd import build
from synth import workload as W
from tests.helpers import oracle_cfg, rand_rows, rand_weights

SOURCE = r"""
#include "%s/kernels.h"
extern "C" int compact(int n, int L) { return dy::compact_form(n, L); }
"""


def test_rule(tmp_path):
    src, so = str(tmp_path / "rule.cpp"), str(tmp_path / "rule.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = C.CDLL(so)
    for L in (1, 5, 6, 77, 513, 1024, 2048, 1 << 30):
        assert lib.compact(0, L)
        # a sweep over all keys behind a loop over this many is slower than the loop over all keys alone
        assert not any(lib.compact(n, L) for n in (L, L - L // 4, -(-L // 4)))
    assert lib.compact(40, 200) and not lib.compact(41, 200)
    assert lib.compact(50, 513) and lib.compact(102, 1024)  # and here it is quicker


MANY = W.LayerShape(hidden=256, n_heads=32, n_kv_heads=32, head_dim=128, ffn=384, dtype="bf16", rope_theta=10000.0)
FEW = W.LayerShape(hidden=256, n_heads=6, n_kv_heads=2, head_dim=128, ffn=384, dtype="bf16", rope_theta=10000.0)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,L,row_lo,first,second", [
    ("many", 192, 0, [38, 39, 192, 0], [39, 0, 1, 192]),  # the line, one more, all, none; and each in another sequence
    ("many", 77, 0, [15, 16, 1], [16, 77, 15]),
    ("few", 640, 0, [128, 129, 640], [0, 128, 300]),   # the keys split over workgroups
    ("few", 200, 120, [40, 41, 80], [80, 0, 40]),      # response steps: the line counts the whole sequence
])
def test_steps_on_both_sides_of_the_line(shape, L, row_lo, first, second):
    import torch
    from paper_2603_08026_amd import binding as Bd
    from paper_2603_08026_amd.layer import Layer
    from tests.helpers import TOL, assert_close
    from tests.test_gpu_layer_step_approx import _round, _teacher_force
    s = MANY if shape == "many" else FEW
    print("forms of the update", shape, L, row_lo, first, second, flush=True)
    cfg, B = oracle_cfg(s), len(first)
    T = B * L
    w = rand_weights(s, 61, bias=True, std=0.08)
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(w)
    x = _round(W.philox(62, "x").standard_normal((B, L, s.hidden), dtype=np.float32), "bf16")
    ref = O.new_caches(B, L, cfg)
    O.full_step(x, w, cfg, ref)
    lay.full_step(lay.upload(x))
    out = Bd.IndexList.empty(T, B)
    for turn, counts in enumerate((first, second)):
        ref = _teacher_force(lay, ref, "bf16")
        idx, off = rand_rows(63 + turn, B, L - row_lo, counts)
        idx = (idx // (L - row_lo) * L + row_lo + idx % (L - row_lo)).astype(idx.dtype)
        x = x.reshape(T, -1).copy()
        x[idx] = W.perturbed_rows(x[idx], np.full(idx.size, 1.0), 65 + turn)
        x = _round(x, "bf16").reshape(B, L, -1)
        O.layer_step_approx(x, idx, w, cfg, ref, -2.0, row_lo=row_lo)
        lay.layer_step_approx(lay.upload(x), lay.make_list(idx, off, cap=T), -2.0, out, None, row_lo)
        torch.cuda.synchronize()
        got = lay.get_caches()
        for name in ("k", "v", "c"):
            assert_close(got[name].reshape(T, -1), ref[name].reshape(T, -1), TOL["bf16"], "step %d: %s" % (turn, name))
    lay.close()
