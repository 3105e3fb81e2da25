"""q|k|v rows that the GEMM's own epilogue finishes (lists with room for at most half of the tokens) against the same rows
through the raw result and the row kernel (a list with room for all tokens): the same plan, sums, bias, rotation and rounding, so
the same bits.  Row counts that leave a last tile of one row, of part of a 16-row block and of a whole one; column tiles of 128, 192
and 256; heads of 128 and 64 columns; tiles and waves that hold queries and keys, or keys and values; sequence lengths that
are no power of two; rows that the list does not name stay as they are."""
import pytest
import torch

from paper_2603_08026_amd import binding as Bd
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
    q1, past, k1, v1 = _refresh(lay, s, x, ids, off, min(n + 11, B * L // 2))
    lay.close()
    assert torch.equal(q1, q0) and torch.equal(k1, k0) and torch.equal(v1, v0)
    assert (past == 3.0).all()
    listed = torch.zeros(B * L, dtype=torch.bool, device="cuda")
    listed[ids.long()] = True
    assert (k1.view(B * L, -1)[~listed] == 5.0).all() and (v1.view(B * L, -1)[~listed] == -7.0).all()
    assert torch.isfinite(q1.float()).all() and not (k1.view(B * L, -1)[listed] == 5.0).all(1).any()
