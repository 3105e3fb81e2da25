"""q|k|v rows that the GEMM's own epilogue finishes (lists with room for at most half of the tokens) against the same rows
through the raw result and the row kernel (a list with room for all tokens): the same plan, sums, bias, rotation and rounding, so
the same bits.  Row counts that leave a last tile of one row, of part of a 16-row block and of a whole one; column tiles of 128, 192
and 256; heads of 128 and 64 columns; tiles and waves that hold queries and keys, or keys and values; sequence lengths that
are no power of two; rows that the list does not name stay as they are."""
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
    "dh64": W.LayerShape(hidden=512, n_heads=18, n_kv_heads=3, head_dim=64, ffn=512, dtype="bf16"),
    "wide": W.LayerShape(hidden=256, n_heads=24, n_kv_heads=12, head_dim=128, ffn=512, dtype="bf16"),
}
CASES = [(s, b, n) for s, b in (("mha", False), ("mha", True), ("gqa", True), ("dh64", True), ("wide", True))
         for n in (129, 257, 300, 513, 1000, 2049, 4085)]


def _cap(n):  # room whose rows the GEMM finishes: a plan made on the host, or from 1100 entries on
    return n + 11 if n < 246 else min(max(n + 11, 1100), 7 * 1171 // 2)


def _refresh(lay, s, x, ids, off, cap):
    buf = torch.zeros(cap, dtype=torch.int32, device="cuda")
    buf[:ids.numel()] = ids
    q = torch.full((cap, s.dq), 3.0, dtype=torch.bfloat16, device="cuda")
    lay.k.fill_(5.0)
    lay.v.fill_(-7.0)
    lay.ctx.qkv_refresh(lay.w, x, Bd.IndexList(buf, off), x.shape[0], x.shape[1], lay.cache, q)
    return q[:ids.numel()].clone(), q[ids.numel():].clone(), lay.k.clone(), lay.v.clone()


@pytest.mark.gpu
@pytest.mark.parametrize("shape,bias,n", CASES)
def test_rows_of_a_list(shape, bias, n):
    from paper_2603_08026_amd.layer import Layer
    s, B, L = SHAPES[shape], 7, 1171
    print("finished q|k|v", shape, bias, n, flush=True)
    g = torch.Generator().manual_seed(n)
    ids = torch.sort(torch.randperm(B * L, generator=g)[:n])[0].to(torch.int32)
    off = torch.tensor([int((ids < b * L).sum()) for b in range(B + 1)], dtype=torch.int32).cuda()
    ids = ids.cuda()
    x = torch.randn(B, L, s.hidden, generator=g).to(torch.bfloat16).cuda()
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(rand_weights(s, 81, bias=bias))
    q0, _, k0, v0 = _refresh(lay, s, x, ids, off, B * L)
    q1, past, k1, v1 = _refresh(lay, s, x, ids, off, _cap(n))
    lay.close()
    assert torch.equal(q1, q0) and torch.equal(k1, k0) and torch.equal(v1, v0)
    assert (past == 3.0).all()
    listed = torch.zeros(B * L, dtype=torch.bool, device="cuda")
    listed[ids.long()] = True
    assert (k1.view(B * L, -1)[~listed] == 5.0).all() and (v1.view(B * L, -1)[~listed] == -7.0).all()
    assert torch.isfinite(q1.float()).all() and not (k1.view(B * L, -1)[listed] == 5.0).all(1).any()


# One list of each of these (hidden 4096, 32 heads; 28 over 4 heads) is full to the counts named: K split by the device (the row kernel finishes
# all rows), not split (the GEMM finishes them), and not split with a last row tile in the weight-streaming tiles (the row
# kernel finishes the rows behind the full tiles).
LISTS = {
    "llada": (W.LayerShape(hidden=4096, n_heads=32, n_kv_heads=32, head_dim=128, ffn=128, dtype="bf16"), 2064),
    "grouped": (W.LayerShape(hidden=3584, n_heads=28, n_kv_heads=4, head_dim=128, ffn=128, dtype="bf16"), 2064),
    "dh64": (W.LayerShape(hidden=1024, n_heads=62, n_kv_heads=1, head_dim=64, ffn=512, dtype="bf16"), 4200),
}
# rows -> (K splits, rows in row tiles) of the plan
COUNTS = {
    "llada": {140: (2, 140), 1281: (1, 1280), 1300: (1, 1280), 1408: (1, 1280), 1409: (1, 1409), 2064: (1, 2064)},
    "grouped": {300: (3, 300), 1600: (1, 1600), 2064: (1, 2064)},
    "dh64": {130: (2, 130), 4097: (1, 4096), 4200: (1, 4096)},
}

SOURCE = r"""
#include "%s/gemm_plan.h"
using namespace dy::mm;
extern "C" int plan(int N, int K, long part_elems, int cap, long tokens, int count, int *out) {
  const PlanArgs a = raw_plan_args(N, K, part_elems, true, 32);
  const GemmPlan p = plan_on_host(a, count);
  out[0] = p.sk; out[1] = p.row_hi;
  return finishing_kernel(few_of_room(true, cap, tokens) || few_results(plan_known(true, cap), cap, N), plan_on_host(a, cap));
}
"""


def test_lists_take_the_kernels_and_plans_they_name(tmp_path):
    src, so = str(tmp_path / "plan.cpp"), str(tmp_path / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = C.CDLL(so)

    def ask(s, cap, tokens, count):
        n, out = s.dq + 2 * s.dkv, (C.c_int * 2)()
        part = max(16 * min(tokens, 2048) * s.dq, tokens * max(n, s.hidden))  # the context's fp32 scratch
        return lib.plan(n, s.hidden, C.c_long(part), cap, C.c_long(tokens), count, out), tuple(out)
    for name, (s, cap) in LISTS.items():
        for count, want in COUNTS[name].items():
            assert ask(s, cap, 2 * cap, count) == (1, want), (name, count)
            assert ask(s, 2 * cap, 2 * cap, count) == (0, want), (name, count)
    for name, _, count in CASES:  # the test above: lists of half the tokens finish their rows in the GEMM, lists of all do not
        cap = _cap(count)
        kernel, (splits, tiled) = ask(SHAPES[name], cap, 7 * 1171, count)
        assert kernel == 1 and splits == 1 and tiled == count, (name, count)
        assert ask(SHAPES[name], 7 * 1171, 7 * 1171, count)[0] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("shape", sorted(LISTS))
def test_one_list_at_several_counts(shape):
    from paper_2603_08026_amd.layer import Layer
    s, cap = LISTS[shape]
    B, L = 4, cap // 2
    g = torch.Generator().manual_seed(85)
    x = torch.randn(B, L, s.hidden, generator=g).to(torch.bfloat16).cuda()
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(rand_weights(s, 86, bias=True))
    for n in COUNTS[shape]:
        print("finished q|k|v of one list", shape, n, flush=True)
        ids = torch.sort(torch.randperm(B * L, generator=g)[:n])[0].to(torch.int32)
        off = torch.tensor([int((ids < b * L).sum()) for b in range(B + 1)], dtype=torch.int32).cuda()
        q0, _, k0, v0 = _refresh(lay, s, x, ids.cuda(), off, B * L)
        q1, past, k1, v1 = _refresh(lay, s, x, ids.cuda(), off, cap)
        assert torch.equal(q1, q0) and torch.equal(k1, k0) and torch.equal(v1, v0), n
        assert (past == 3.0).all(), n
        listed = torch.zeros(B * L, dtype=torch.bool, device="cuda")
        listed[ids.long().cuda()] = True
        assert (k1.view(B * L, -1)[~listed] == 5.0).all() and (v1.view(B * L, -1)[~listed] == -7.0).all(), n
        assert torch.isfinite(q1.float()).all() and not (k1.view(B * L, -1)[listed] == 5.0).all(1).any(), n
    lay.close()
