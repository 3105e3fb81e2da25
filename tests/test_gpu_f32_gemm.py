"""fp32 GEMMs on the matrix instructions: row counts at the edges of the 16- and 32-row tiles, capacities on
both sides of the one that changes the tile, a K of two wave steps (two of the four waves have none) and one
of five.  Against the oracle at 1e-5: sums of at most 320 products of order 1 in fp32, 2^-24 * sqrt(320) with
an order of magnitude to spare."""
import numpy as np
import pytest
import torch

from tests.helpers import assert_close, oracle_cfg, rand_rows, rand_weights
from oracle import dyllm_oracle as O
from paper_2603_08026_amd.layer import Layer, to_device, to_host
from synth import workload as W

pytestmark = pytest.mark.gpu

SHAPE = W.LayerShape(hidden=128, n_heads=4, n_kv_heads=2, head_dim=64, ffn=320, dtype="f32")


@pytest.mark.parametrize("count,cap", [(0, 40), (1, 1), (15, 16), (16, 17), (17, 40), (31, 600), (33, 600), (600, 600)])
def test_f32_rows_and_tiles(count, cap):
    print("f32 gemm", count, cap, flush=True)
    B, L = 2, 320
    T = B * L
    cfg = oracle_cfg(SHAPE)
    lay = Layer.from_shape(SHAPE, B, L)
    w = rand_weights(SHAPE, 61, bias=True)
    lay.set_weights(w)
    idx, off = rand_rows(62, B, L, [count - count // 2, count // 2])
    rows = lay.make_list(idx, off, cap=cap)
    x, c, out0 = (W.philox(63, n).standard_normal((T, d), dtype=np.float32)
                  for n, d in (("x", SHAPE.hidden), ("c", SHAPE.dq), ("o", SHAPE.hidden)))
    ref = out0.astype(np.float64)
    O.salient_ffn(x, c, idx, w, cfg, ref)
    d_out = to_device(out0, "f32")
    lay.ctx.salient_ffn(lay.w, to_device(x, "f32"), to_device(c, "f32"), rows, B, L, d_out)
    q_out = torch.zeros(cap, SHAPE.dq, device="cuda")
    lay.ctx.qkv_refresh(lay.w, lay.upload(x.reshape(B, L, -1)), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    others = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    if count:
        assert_close(got[idx], ref[idx], 1e-5, "ffn rows")
        q, k, v = O.project_qkv(O.rmsnorm(x[idx], w["g_attn"], cfg.rms_eps), idx % L, w, cfg)
        assert_close(to_host(q_out)[:count], q.reshape(count, -1), 1e-5, "q")
        assert_close(to_host(lay.k).reshape(T, -1)[idx], k.reshape(count, -1), 1e-5, "k")
        assert_close(to_host(lay.v).reshape(T, -1)[idx], v.reshape(count, -1), 1e-5, "v")
    lay.close()
