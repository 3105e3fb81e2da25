"""Rows of every width that the row kernels tell apart, against the oracle."""
import numpy as np
import pytest
import torch

from tests.helpers import assert_close, oracle_cfg, rand_rows, rand_weights
from oracle import dyllm_oracle as O
from paper_2603_08026_amd.layer import Layer, to_device, to_host
from synth import workload as W

pytestmark = pytest.mark.gpu


# A thread of the norm has one or two vectors of a row, the second perhaps of fewer threads (hidden 128, 2048, 2176, 3968, 4096), or up to four
# (4224, 8192), or the workgroup is the wide one (8320); rows listed with and without a plan to make, few enough that K is
# split and the row kernel behind sums, rotates and merges four elements at a time, and known ones.  bf16 results: 2e-2 as everywhere.
@pytest.mark.parametrize("hidden", [128, 2048, 2176, 3968, 4096, 4224, 8192, 8320])
@pytest.mark.parametrize("kv,dh,bias", [(2, 64, True), (1, 128, False)])
def test_norm_and_projection(hidden, kv, dh, bias):
    print("row width", hidden, kv, dh, bias, flush=True)
    s = W.LayerShape(hidden=hidden, n_heads=2, n_kv_heads=kv, head_dim=dh, ffn=128, dtype="bf16")
    cfg = oracle_cfg(s)
    B, L = 2, 200
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 91, bias=bias)
    lay.set_weights(w)
    x = W.round_bf16(W.philox(92, "x").standard_normal((B, L, hidden), dtype=np.float32))
    for counts, cap in (([3, 1], 4), ([90, 61], 260), ([150, 180], 330)):
        idx, off = rand_rows(93, B, L, counts)
        k0, v0 = (W.round_bf16(W.philox(94, n).standard_normal((B * L, s.dkv), dtype=np.float32)) for n in "kv")
        lay.k.copy_(to_device(k0, "bf16").view_as(lay.k))
        lay.v.copy_(to_device(v0, "bf16").view_as(lay.v))
        rows = lay.make_list(idx, off, cap=cap)
        q_out = torch.zeros(cap, s.dq, dtype=torch.bfloat16, device="cuda")
        lay.ctx.qkv_refresh(lay.w, lay.upload(x), rows, B, L, lay.cache, q_out)
        torch.cuda.synchronize()
        q, k, v = O.project_qkv(O.rmsnorm(x.reshape(B * L, -1)[idx], w["g_attn"], cfg.rms_eps), idx % L, w, cfg)
        assert_close(to_host(q_out)[:idx.size], q.reshape(idx.size, -1), 2e-2, "q")
        kg, vg = to_host(lay.k).reshape(B * L, -1), to_host(lay.v).reshape(B * L, -1)
        assert_close(kg[idx], k.reshape(idx.size, -1), 2e-2, "k rows")
        assert_close(vg[idx], v.reshape(idx.size, -1), 2e-2, "v rows")
        others = np.setdiff1d(np.arange(B * L), idx)
        assert np.array_equal(kg[others], k0[others].astype(np.float64)) and np.array_equal(vg[others], v0[others].astype(np.float64))
        assert np.all(to_host(q_out)[idx.size:] == 0)
    lay.close()


# fp32: the norm kernel runs ahead of the candidates' GEMM of the approximate step and where a result takes the place of x; one or two
# vectors a thread (2048), up to four (2112, 4096), the wide workgroup (4160).  Sums of up to 4160 products in fp32, 2^-24 * sqrt(4160) = 4e-6 of their size: 1e-4 as
# everywhere.
@pytest.mark.parametrize("hidden", [64, 2048, 2112, 4096, 4160])
@pytest.mark.parametrize("counts", [[3, 1], [90, 61]])
def test_norm_and_projection_f32(hidden, counts):
    print("fp32 row width", hidden, counts, flush=True)
    s = W.LayerShape(hidden=hidden, n_heads=2, n_kv_heads=1, head_dim=64, ffn=128, dtype="f32")
    cfg = oracle_cfg(s)
    B, L = 2, 100
    w = rand_weights(s, 95, bias=True)
    x = W.philox(96, "x").standard_normal((B, L, hidden), dtype=np.float32)
    idx, off = rand_rows(97, B, L, counts)
    q, k, v = O.project_qkv(O.rmsnorm(x.reshape(B * L, -1)[idx], w["g_attn"], cfg.rms_eps), idx % L, w, cfg)
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(w)
    rows = lay.make_list(idx, off)
    # q in the place of x (whose rows are the wider ones, or hold all of q between them)
    room = torch.zeros(max(B * L * hidden, idx.size * s.dq), device="cuda")
    xd = room[:B * L * hidden].view(B, L, hidden)
    xd.copy_(torch.from_numpy(x))
    lay.ctx.qkv_refresh(lay.w, xd, rows, B, L, lay.cache, room)
    torch.cuda.synchronize()
    assert_close(to_host(room[:idx.size * s.dq]), q.reshape(-1), 1e-4, "q in the place of x")
    assert_close(to_host(lay.k).reshape(B * L, -1)[idx], k.reshape(idx.size, -1), 1e-4, "k rows")
    # candidates of the approximate step, which also takes q of all tokens
    lay.k.zero_()
    lay.v.zero_()
    lay.c.copy_(torch.randn(lay.c.shape, generator=torch.Generator().manual_seed(5)))
    lay.layer_step_approx(lay.upload(x), rows, 0.5)
    torch.cuda.synchronize()
    assert_close(to_host(lay.k).reshape(B * L, -1)[idx], k.reshape(idx.size, -1), 1e-4, "candidates' k")
    assert_close(to_host(lay.v).reshape(B * L, -1)[idx], v.reshape(idx.size, -1), 1e-4, "candidates' v")
    lay.close()
