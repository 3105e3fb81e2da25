"""Attention kernels at the edges of their tiles, against the oracle."""
import numpy as np
import pytest
import torch

from tests.helpers import assert_close, rand_rows
from oracle import dyllm_oracle as O
from paper_2603_08026_amd.layer import Layer, to_device, to_host
from synth import workload as W

pytestmark = pytest.mark.gpu


def _partial(shape, B, L, counts, tol, cap):
    idx, off = rand_rows(71, B, L, counts)
    M = idx.size
    def vals(name, *sh):
        return W.philox(72, name).standard_normal(sh, dtype=np.float32)
    q, k, v = vals("q", M, shape.n_heads, shape.head_dim), vals("k", B, L, shape.n_kv_heads, shape.head_dim), vals("v", B, L, shape.n_kv_heads, shape.head_dim)
    lay = Layer.from_shape(shape, B, L)
    rows = lay.make_list(idx, off, cap=cap)
    out, qd = torch.full((cap, shape.dq), -7.0, device="cuda"), torch.full((cap, shape.dq), float("nan"), device="cuda")
    qd[:M] = to_device(q.reshape(M, -1), "f32")
    lay.ctx.partial_attention(qd, to_device(k, "f32"), to_device(v, "f32"), rows, B, L, out)
    torch.cuda.synchronize()
    assert_close(to_host(out)[:M], O.partial_attention(q, k, v, idx, B, L), tol, "context rows")
    assert (out[M:] == -7.0).all()  # entries that the list has room for and does not hold
    lay.close()


# fp32: 16-row query tiles, 32-key tiles, one or several to a key split; lists that are full and that have room for every
# token, whose surplus tiles do not exist.  Sums of at most 128 products and 200 weights in fp32: 2^-24 * sqrt(200) =
# 8e-7, an order of magnitude to spare.
@pytest.mark.parametrize("spare", [False, True])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("L,counts", [(1, [1]), (31, [16]), (32, [17]), (33, [15, 33]), (64, [1, 0]), (97, [40, 16]), (200, [3])])
def test_f32_attention(dh, L, counts, spare):
    print("f32 attention", dh, L, counts, spare, flush=True)
    s = W.LayerShape(hidden=128, n_heads=4, n_kv_heads=2, head_dim=dh, ffn=192, dtype="f32")
    _partial(s, len(counts), L, counts, 1e-5, len(counts) * L if spare else sum(counts))
