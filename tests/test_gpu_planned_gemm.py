"""GEMM plans made on the device: lists whose capacity says nothing about their count, as the generation
loop carries them.  Counts at the edges of the regimes (weight streaming up to 128 rows, 256-row tiles, a
short last row tile), a K of 26 slices (K splits that differ by a slice), and capacities on both sides of
the one above which the down projection always gets its sum kernel.  Against the oracle, at the bars of
every other bf16 layer tensor."""
import numpy as np
import pytest
import torch

from tests.helpers import TOL, assert_close, oracle_cfg, rand_rows, rand_weights
from oracle import dyllm_oracle as O
from paper_2603_08026_amd.layer import Layer, to_device, to_host
from synth import workload as W

pytestmark = pytest.mark.gpu

SHAPE = W.LayerShape(hidden=1024, n_heads=8, n_kv_heads=2, head_dim=128, ffn=1664, dtype="bf16")


def _vals(seed, shape):
    return W.round_bf16(W.philox(seed, "planned").standard_normal(shape, dtype=np.float32))


@pytest.fixture(scope="module")
def layer():
    lay = Layer.from_shape(SHAPE, 3, 1400)  # (the largest list: 4200 entries)
    w = rand_weights(SHAPE, 51, bias=True)
    lay.set_weights(w)
    yield lay, w
    lay.close()


@pytest.mark.parametrize("cap", [1000, 4200])
@pytest.mark.parametrize("count", [0, 1, 127, 128, 129, 256, 257, 330, 384, 385, 640])
def test_count_far_below_capacity(layer, count, cap):
    print("planned gemm", count, cap, flush=True)
    lay, w = layer
    B, L, T = 3, 1400, 4200
    cfg = oracle_cfg(SHAPE)
    per = [count // B + (1 if b < count % B else 0) for b in range(B)]
    idx, off = rand_rows(52, B, L, per)
    rows = lay.make_list(idx, off, cap=cap)
    x, c, out0 = _vals(53, (T, SHAPE.hidden)), _vals(54, (T, SHAPE.dq)), _vals(55, (T, SHAPE.hidden))

    # the FFN half: out-projection, gate|up, down
    ref = out0.astype(np.float64)
    O.salient_ffn(x, c, idx, w, cfg, ref)
    d_out = to_device(out0, "bf16")
    lay.ctx.salient_ffn(lay.w, to_device(x, "bf16"), to_device(c, "bf16"), rows, B, L, d_out)
    # q/k/v
    q_out = torch.zeros(cap, SHAPE.dq, dtype=torch.bfloat16, device="cuda")
    lay.k.zero_()
    lay.v.zero_()
    lay.ctx.qkv_refresh(lay.w, lay.upload(x.reshape(B, L, -1)), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    others = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    kg, vg = to_host(lay.k).reshape(T, -1), to_host(lay.v).reshape(T, -1)
    assert not kg[others].any() and not vg[others].any()
    if count:
        assert_close(got[idx], ref[idx], TOL["bf16"], "ffn rows")
        n = O.rmsnorm(x[idx], w["g_attn"], cfg.rms_eps)
        q, k, v = O.project_qkv(n, idx % L, w, cfg)
        assert_close(to_host(q_out)[:count], q.reshape(count, -1), TOL["bf16"], "q")
        assert_close(kg[idx], k.reshape(count, -1), TOL["bf16"], "k")
        assert_close(vg[idx], v.reshape(count, -1), TOL["bf16"], "v")
