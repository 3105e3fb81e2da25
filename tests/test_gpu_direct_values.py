"""Values that the q|k|v GEMM of a dense step of many rows writes itself, against the same tokens given as a list, whose
values go through the row kernel: the same sums, bias and rounding, so the same bits.  Row counts at the edge of that
rule and with a last tile of one row and of part of a 16-row block; value columns that start inside a column tile and
inside a wave's 128 columns of it."""
import pytest
import torch

from paper_2603_08026_amd import binding as Bd
from paper_2603_08026_amd.layer import Layer
from synth import workload as W
from tests.helpers import rand_weights

pytestmark = pytest.mark.gpu

SHAPES = {
    "mha": W.LayerShape(hidden=512, n_heads=8, n_kv_heads=8, head_dim=128, ffn=512, dtype="bf16"),
    "gqa": W.LayerShape(hidden=512, n_heads=7, n_kv_heads=1, head_dim=128, ffn=512, dtype="bf16"),
    "dh64": W.LayerShape(hidden=512, n_heads=16, n_kv_heads=1, head_dim=64, ffn=512, dtype="bf16"),
}


@pytest.mark.parametrize("shape,bias", [("mha", False), ("mha", True), ("gqa", True), ("dh64", True)])
@pytest.mark.parametrize("B,L", [(2, 2048), (1, 4097), (3, 1367), (5, 1024)])
def test_values_of_a_dense_step(shape, bias, B, L):
    s = SHAPES[shape]
    print("direct values", shape, bias, B, L, flush=True)
    T = B * L
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(rand_weights(s, 81, bias=bias))
    x = torch.randn(B, L, s.hidden, generator=torch.Generator().manual_seed(82)).to(torch.bfloat16).cuda()
    every = Bd.IndexList(torch.arange(T, dtype=torch.int32, device="cuda"),
                         torch.arange(B + 1, dtype=torch.int32, device="cuda") * L)
    q = torch.zeros(T, s.dq, dtype=torch.bfloat16, device="cuda")
    lay.ctx.qkv_refresh(lay.w, x, every, B, L, lay.cache, q)
    k, v = lay.k.clone(), lay.v.clone()
    lay.k.zero_()
    lay.v.fill_(float("nan"))
    lay.full_step(x)
    assert torch.equal(lay.v, v) and torch.equal(lay.k, k)
    lay.close()
