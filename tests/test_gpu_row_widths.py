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
