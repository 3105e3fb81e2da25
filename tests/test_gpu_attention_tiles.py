"""Attention kernels at the edges of their tiles, against the oracle."""
import numpy as np
import pytest
import torch

from tests.helpers import assert_close, rand_rows
from oracle import dyllm_oracle as O
from paper_2603_08026_amd.layer import Layer, to_device, to_host
from synth import workload as W

pytestmark = pytest.mark.gpu


def _partial(shape, B, L, counts, tol, cap=None):
    idx, off = rand_rows(71, B, L, counts)
    M, dt = idx.size, shape.dtype
    def vals(name, *sh):
        a = W.philox(72, name).standard_normal(sh, dtype=np.float32)
        return W.round_bf16(a) if dt == "bf16" else a
    q, k, v = vals("q", M, shape.n_heads, shape.head_dim), vals("k", B, L, shape.n_kv_heads, shape.head_dim), vals("v", B, L, shape.n_kv_heads, shape.head_dim)
    lay = Layer.from_shape(shape, B, L)
    cap = M if cap is None else cap
    rows = lay.make_list(idx, off, cap=cap)
    out, qd = (torch.zeros(cap, n, dtype=lay.k.dtype, device="cuda") for n in (shape.dq, shape.dq))
    qd[:M] = to_device(q.reshape(M, -1), dt)
    lay.ctx.partial_attention(qd, to_device(k, dt), to_device(v, dt), rows, B, L, out)
    torch.cuda.synchronize()
    assert_close(to_host(out)[:M], O.partial_attention(q, k, v, idx, B, L), tol, "context rows")
    assert not to_host(out)[M:].any()
    lay.close()


# fp32: 16-row query tiles, 32-key tiles, one or several to a key split.  Sums of at most 128 products and 200 weights in
# fp32: 2^-24 * sqrt(200) = 8e-7, an order of magnitude to spare.
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("L,counts", [(1, [1]), (31, [16]), (32, [17]), (33, [15, 33]), (64, [1, 0]), (97, [40, 16]), (200, [3])])
def test_f32_attention(dh, L, counts):
    print("f32 attention", dh, L, counts, flush=True)
    s = W.LayerShape(hidden=128, n_heads=4, n_kv_heads=2, head_dim=dh, ffn=192, dtype="f32")
    _partial(s, len(counts), L, counts, 1e-5)
