"""The approximate step at head_dim 128, whose normalisers come from a sweep over all keys beside the compact candidates:
candidate counts around the key tiles (none, one, a tile, one more), sequence lengths around the two tiles that a step
of the sweep takes, and few heads (the keys split over workgroups) and many."""
import numpy as np
import pytest

from oracle import dyllm_oracle as O
from paper_2603_08026_amd.layer import Layer
from synth import workload as W
from tests.helpers import oracle_cfg, rand_rows, rand_weights
from tests.test_gpu_layer_step_approx import _check_step, _round, _teacher_force

pytestmark = pytest.mark.gpu

FEW = W.LayerShape(hidden=256, n_heads=4, n_kv_heads=1, head_dim=128, ffn=384, dtype="bf16", rope_theta=10000.0)
MANY = W.LayerShape(hidden=256, n_heads=32, n_kv_heads=32, head_dim=128, ffn=384, dtype="bf16", rope_theta=10000.0)


@pytest.mark.parametrize("shape,L,counts", [
    ("few", 64, [0, 1, 32]), ("few", 65, [33, 0, 64]), ("few", 127, [31, 127, 2]), ("few", 513, [1, 160, 0]),
    ("many", 193, [0, 33, 65]), ("many", 320, [129, 1, 0]), ("many", 31, [31, 3, 0]),
])
def test_candidates_and_lengths(shape, L, counts):
    s = FEW if shape == "few" else MANY
    print("approx normaliser", shape, L, counts, flush=True)
    cfg, B = oracle_cfg(s), len(counts)
    T = B * L
    w = rand_weights(s, 91, bias=True, std=0.08)
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(w)
    x0 = _round(W.philox(92, "x0").standard_normal((B, L, s.hidden), dtype=np.float32), "bf16")
    ref = O.new_caches(B, L, cfg)
    O.full_step(x0, w, cfg, ref)
    lay.full_step(lay.upload(x0))
    ref = _teacher_force(lay, ref, "bf16")
    idx, off = rand_rows(93, B, L, counts)
    x1 = x0.copy().reshape(T, -1)
    x1[idx] = W.perturbed_rows(x1[idx], np.full(idx.size, 1.0), 94)
    x1 = _round(x1, "bf16").reshape(B, L, -1)
    probe = O.layer_step_approx(x1, idx, w, cfg, {k: v.copy() for k, v in ref.items()}, 0.5)[2]
    _check_step(lay, ref, w, cfg, x1, idx, off, float(np.quantile(probe, 0.3)), "step")
    lay.close()


# Scores that spread over many powers of two (W_q four times as large): for most queries the best key is no candidate and lies
# more than 2^8 above all of them, so that the sweep over all keys moves the reference of a sum of P V that is not zero.
# Against float32 attention over the queries, keys and values that the layer itself stores (bf16), so that the spread does
# not multiply the rounding of q: a context is rounded once (2^-9 of itself), probabilities and residuals to bf16.
@pytest.mark.parametrize("shape,L,counts,nan_at", [
    ("few", 300, [3, 1, 0], None), ("many", 257, [2, 4, 9], None), ("few", 700, [2, 130, 5], None),
    ("many", 200, [3, 2, 1], (1, 77)), ("few", 300, [3, 2, 1], (1, 10)),  # a query of NaN: its own row alone
])
def test_best_key_is_no_candidate(shape, L, counts, nan_at):
    import torch
    from paper_2603_08026_amd import binding as Bd
    s = FEW if shape == "few" else MANY
    print("approx normaliser, spread scores", shape, L, counts, nan_at, flush=True)
    B, H, dh, g = len(counts), s.n_heads, s.head_dim, s.n_heads // s.n_kv_heads
    T = B * L
    w = rand_weights(s, 101, std=0.08)
    w["wq"] = 4.0 * w["wq"]
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(w)
    x0 = _round(W.philox(102, "x0").standard_normal((B, L, s.hidden), dtype=np.float32), "bf16")
    lay.full_step(lay.upload(x0))
    idx, off = rand_rows(103, B, L, counts)
    x1 = x0.copy().reshape(T, -1)
    x1[idx] = W.perturbed_rows(x1[idx], np.full(idx.size, 1.0), 104)
    if nan_at is not None:
        assert nan_at[0] * L + nan_at[1] not in idx
        x1[nan_at[0] * L + nan_at[1]] = np.nan
    x1 = _round(x1, "bf16").reshape(B, L, -1)
    old_v, old_c = lay.v.float().clone(), lay.c.float().clone()
    k0, v0 = lay.k.clone(), lay.v.clone()
    every = Bd.IndexList(torch.arange(T, dtype=torch.int32, device="cuda"), torch.arange(B + 1, dtype=torch.int32, device="cuda") * L)
    q = torch.zeros(T, s.dq, dtype=torch.bfloat16, device="cuda")
    lay.ctx.qkv_refresh(lay.w, lay.upload(x1), every, B, L, lay.cache, q)
    lay.k.copy_(k0)
    lay.v.copy_(v0)
    lay.layer_step_approx(lay.upload(x1), lay.make_list(idx, off), -2.0, Bd.IndexList.empty(T, B))
    torch.cuda.synchronize()
    dv = (lay.v.float() - old_v).to(torch.bfloat16).float().cpu()
    k, q, c0, c1 = lay.k.float().cpu(), q.float().cpu().view(B, L, H, dh), old_c.cpu().view(B, L, H, dh), lay.c.float().cpu().view(B, L, H, dh)
    moved = total = 0
    for b in range(B):
        cand = torch.from_numpy(idx[off[b]:off[b + 1]].astype(np.int64) - b * L)
        others = torch.ones(L, dtype=torch.bool)
        others[cand] = False
        for h in range(H):
            sc = q[b, :, h] @ k[b, :, h // g].t() / dh ** 0.5
            want = c0[b, :, h] + torch.softmax(sc, -1)[:, cand] @ dv[b, cand, h // g]
            live = others.clone()
            if nan_at is not None and nan_at[0] == b:
                live[nan_at[1]] = False
                assert torch.isnan(c1[b, nan_at[1], h]).all()
            if len(cand):
                moved += int((sc[live].max(-1)[0] - sc[live][:, cand].max(-1)[0] > 8 * np.log(2)).sum())
                total += int(live.sum())
            err = float((c1[b, live, h] - want[live]).abs().max() / c0[b].nan_to_num().abs().max())
            assert err < 1e-2, (b, h, err)
    assert moved > total // 4
    lay.close()
