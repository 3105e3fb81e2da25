"""Keys and values that the q|k|v GEMM of a dense step writes itself, against the same tokens given as a list, which go through
the row kernel: the same sums, bias, rotation and rounding, so the same bits.  Few and many rows, row counts with a last tile of one row and of part of a 16-row block; value columns that start at a column tile, at a wave's
columns, and inside them (192- and 256-column tiles); a last row tile that goes to the weight-streaming tiles, whose values the
row kernel finishes; NaN and infinities.  The plans that the cases name are checked on the CPU."""
import ctypes as C
import subprocess

import pytest
import torch

from paper_2603_08026_amd import binding as Bd
from paper_2603_08026_amd import build
from synth import workload as W
from tests.helpers import rand_weights

SHAPES = {
    "mha": W.LayerShape(hidden=512, n_heads=8, n_kv_heads=8, head_dim=128, ffn=512, dtype="bf16"),
    "gqa": W.LayerShape(hidden=512, n_heads=7, n_kv_heads=1, head_dim=128, ffn=512, dtype="bf16"),
    "dh64": W.LayerShape(hidden=512, n_heads=16, n_kv_heads=1, head_dim=64, ffn=512, dtype="bf16"),
    "inside": W.LayerShape(hidden=512, n_heads=46, n_kv_heads=1, head_dim=64, ffn=512, dtype="bf16"),
    "streamed": W.LayerShape(hidden=1024, n_heads=62, n_kv_heads=1, head_dim=64, ffn=512, dtype="bf16"),
}
# shape, B, L -> columns of a tile, rows in row tiles (one K split in all: rows are finished)
PLANS = {
    ("mha", 2, 2048): (192, 4096), ("mha", 1, 4097): (256, 4097), ("mha", 3, 1367): (256, 4101), ("mha", 5, 1024): (256, 5120),
    ("gqa", 2, 2048): (128, 4096), ("gqa", 1, 4097): (128, 4097), ("gqa", 3, 1367): (128, 4101), ("gqa", 5, 1024): (128, 5120),
    ("dh64", 2, 2048): (128, 4096), ("dh64", 1, 4097): (128, 4097), ("dh64", 3, 1367): (128, 4101), ("dh64", 5, 1024): (128, 5120),
    # first value column 3008: in the last 64 of a wave's 192, and 64 into a wave's 128
    ("inside", 2, 2048): (192, 4096), ("inside", 1, 4097): (256, 4097), ("inside", 3, 1367): (256, 4101),
    ("streamed", 1, 4097): (256, 4096), ("streamed", 3, 1400): (256, 4096),
    # few rows, in tiles of 32 rows and more; a last row tile of one row in the streaming tiles
    ("mha", 1, 129): (128, 129), ("mha", 1, 300): (128, 300), ("mha", 2, 512): (128, 1024), ("mha", 3, 683): (128, 2049),
    ("gqa", 1, 129): (128, 129), ("gqa", 3, 683): (128, 2049), ("dh64", 1, 300): (128, 300), ("dh64", 2, 512): (128, 1024),
    ("inside", 1, 257): (128, 257), ("inside", 2, 1500): (256, 3000), ("streamed", 3, 683): (128, 2048),
}
CASES = [(s, b, *bl) for s, b in (("mha", False), ("mha", True), ("gqa", True), ("dh64", True))
         for bl in ((2, 2048), (1, 4097), (3, 1367), (5, 1024))]
CASES += [("inside", True, 2, 2048), ("inside", True, 1, 4097), ("inside", True, 3, 1367), ("streamed", True, 1, 4097),
          ("streamed", True, 3, 1400)]
CASES += [(s, True, B, L) for s, B, L in PLANS if B * L < 4096]

SOURCE = r"""
#include "%s/gemm_plan.h"
using namespace dy::mm;
extern "C" void plan(int N, int K, long part_elems, int M, int *out) {
  const GemmPlan p = plan_on_host(raw_plan_args(N, K, part_elems, true, 32), M);
  out[0] = p.xl == PLAN_X ? 256 : p.xl == PLAN_W ? 192 : 128;
  out[1] = p.row_hi; out[2] = p.sk; out[3] = finishing_kernel(false, p);
}
"""


def test_cases_run_the_plans_they_name(tmp_path):
    src, so = str(tmp_path / "plan.cpp"), str(tmp_path / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = C.CDLL(so)
    inside = set()
    for shape, _, B, L in CASES:
        s, T, out = SHAPES[shape], B * L, (C.c_int * 4)()
        n = s.dq + 2 * s.dkv
        part = max(16 * min(T, 2048) * s.dq, T * max(n, s.hidden))  # the context's fp32 scratch
        lib.plan(n, s.hidden, C.c_long(part), T, out)
        assert (out[0], out[1]) == PLANS[shape, B, L] and out[2] == 1 and out[3], (shape, T, tuple(out))
        wave = {128: 64, 192: 192, 256: 128}[out[0]]
        if (s.dq + s.dkv) % wave:
            inside.add(out[0])
    assert inside == {192, 256}  # (a wave's 64 columns of a 128-column tile are a run of their own)


def _both(s, B, L, weights, x):
    """(keys, values) through the list and of the dense step."""
    from paper_2603_08026_amd.layer import Layer
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(weights)
    every = Bd.IndexList(torch.arange(B * L, dtype=torch.int32, device="cuda"),
                         torch.arange(B + 1, dtype=torch.int32, device="cuda") * L)
    q = torch.zeros(B * L, s.dq, dtype=torch.bfloat16, device="cuda")
    lay.ctx.qkv_refresh(lay.w, x, every, B, L, lay.cache, q)
    listed = lay.k.clone(), lay.v.clone()
    lay.k.zero_()
    lay.v.fill_(-7.0)
    lay.full_step(x)
    dense = lay.k.clone(), lay.v.clone()
    lay.close()
    return listed, dense


@pytest.mark.gpu
@pytest.mark.parametrize("shape,bias,B,L", CASES)
def test_values_of_a_dense_step(shape, bias, B, L):
    s = SHAPES[shape]
    print("direct values", shape, bias, B, L, flush=True)
    x = torch.randn(B, L, s.hidden, generator=torch.Generator().manual_seed(82)).to(torch.bfloat16).cuda()
    (k0, v0), (k1, v1) = _both(s, B, L, rand_weights(s, 81, bias=bias), x)
    assert torch.equal(v1, v0) and torch.equal(k1, k0)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,B,L", [("inside", 1, 4097), ("streamed", 1, 4097)])
def test_nan_and_infinities_stay_in_their_rows_and_columns(shape, B, L):
    s = SHAPES[shape]
    print("direct values, not finite", shape, flush=True)
    w = rand_weights(s, 83, bias=True)
    w["bv"][3], w["bv"][17], w["bv"][40] = float("inf"), float("-inf"), float("nan")
    x = torch.randn(B, L, s.hidden, generator=torch.Generator().manual_seed(84)).to(torch.bfloat16).cuda()
    rows = [0, 15, 1000, L - 1]
    x[0, rows, 5] = float("nan")
    (k0, v0), (k1, v1) = _both(s, B, L, w, x)
    assert torch.equal(torch.isnan(v1), torch.isnan(v0)) and torch.equal(torch.nan_to_num(v1), torch.nan_to_num(v0))
    v = v1.view(L, -1)
    clean = torch.ones(L, dtype=torch.bool, device="cuda")
    clean[rows] = False
    assert torch.isnan(v[rows]).all()
    assert (v[clean, 3] == float("inf")).all() and (v[clean, 17] == float("-inf")).all() and torch.isnan(v[clean, 40]).all()
    cols = torch.ones(s.dkv, dtype=torch.bool, device="cuda")
    cols[[3, 17, 40]] = False
    assert torch.isfinite(v[clean][:, cols]).all()
