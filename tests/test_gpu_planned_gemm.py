"""GEMM plans made on the device: lists whose capacity says nothing about their count, as the generation
loop carries them.  Counts at the edges of the regimes (weight streaming up to 128 rows, 256-row tiles, a
short last row tile), a K of 26 slices (K splits that differ by a slice), and capacities below, inside and above
the range in which the down projection has neither a K split nor a sum kernel; and the plans of REGIMES.  Against the
oracle, at the bars of every other bf16 layer tensor.  test_gemm_plan_host.py checks that the cases are planned as
they say."""
import numpy as np
import pytest
import torch

from tests.helpers import TOL, assert_close, oracle_cfg, rand_rows, rand_weights
from oracle import dyllm_oracle as O
from paper_2603_08026_amd.layer import Layer, to_device, to_host
from synth import workload as W

pytestmark = pytest.mark.gpu

SHAPE = W.LayerShape(hidden=1024, n_heads=8, n_kv_heads=2, head_dim=128, ffn=1664, dtype="bf16")
NO_SUMS_CAP = 2600  # full, the list would not split the down projection's (short) K: no sum kernel, no split for any count
WIDE = W.LayerShape(hidden=4096, n_heads=32, n_kv_heads=16, head_dim=128, ffn=12288, dtype="bf16")
SHORT_K = W.LayerShape(hidden=4096, n_heads=32, n_kv_heads=8, head_dim=128, ffn=2048, dtype="bf16")

# (layer, rows, capacity of their list, {GEMM: (columns of the row tiles, K splits, rows in row tiles, splits of the
# streamed rows behind them)})
REGIMES = [
    # row tiles of 256 x 256 with split sums, and streamed rows with another number of them
    (WIDE, 1290, 1290, {"down": (256, 3, 1280, 4), "gate_up": (256, 1, 1280, 1), "oproj": (256, 2, 1290, 1)}),
    (WIDE, 1290, 2100, {"down": (256, 3, 1280, 4), "gate_up": (256, 1, 1280, 1), "oproj": (256, 2, 1290, 1)}),
    # q|k|v and out-projection: whole sums in the row tiles, split ones in the streamed rows
    (WIDE, 2075, 2100, {"qkv": (256, 1, 2048, 2), "oproj": (128, 1, 2048, 4), "down": (256, 2, 2048, 4)}),
    # down projection finished by its own epilogue up to row 4096, streamed rows summed behind it
    (SHORT_K, 4129, 4200, {"down": (256, 1, 4096, 4)}),
    # ... and finished in all rows: the sum kernel finds nothing to do
    (SHAPE, 2600, 4200, {"down": (128, 1, 2600, 1)}),
    # a few rows in a list that needs no split when it is full
    (WIDE, 330, 3000, {"down": (128, 4, 330, 1)}),
]


def _vals(seed, shape):
    return W.round_bf16(W.philox(seed, "planned").standard_normal(shape, dtype=np.float32))


@pytest.fixture(scope="module")
def layer():
    lay = Layer.from_shape(SHAPE, 3, 1400)  # (the largest list: 4200 entries)
    w = rand_weights(SHAPE, 51, bias=True)
    lay.set_weights(w)
    yield lay, w
    lay.close()


def _check(lay, w, shape, B, L, count, cap):
    T = B * L
    cfg = oracle_cfg(shape)
    per = [count // B + (1 if b < count % B else 0) for b in range(B)]
    idx, off = rand_rows(52, B, L, per)
    rows = lay.make_list(idx, off, cap=cap)
    x, c, out0 = _vals(53, (T, shape.hidden)), _vals(54, (T, shape.dq)), _vals(55, (T, shape.hidden))

    # the FFN half: out-projection, gate|up, down
    ref = out0.astype(np.float64)
    O.salient_ffn(x, c, idx, w, cfg, ref)
    d_out = to_device(out0, "bf16")
    lay.ctx.salient_ffn(lay.w, to_device(x, "bf16"), to_device(c, "bf16"), rows, B, L, d_out)
    # q/k/v
    q_out = torch.zeros(cap, shape.dq, dtype=torch.bfloat16, device="cuda")
    lay.k.zero_()
    lay.v.zero_()
    lay.ctx.qkv_refresh(lay.w, lay.upload(x.reshape(B, L, -1)), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    others = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    kg, vg = to_host(lay.k).reshape(T, -1), to_host(lay.v).reshape(T, -1)
    assert not kg[others].any() and not vg[others].any()
    assert not to_host(q_out)[count:].any()
    if count:
        assert_close(got[idx], ref[idx], TOL["bf16"], "ffn rows")
        n = O.rmsnorm(x[idx], w["g_attn"], cfg.rms_eps)
        q, k, v = O.project_qkv(n, idx % L, w, cfg)
        assert_close(to_host(q_out)[:count], q.reshape(count, -1), TOL["bf16"], "q")
        assert_close(kg[idx], k.reshape(count, -1), TOL["bf16"], "k")
        assert_close(vg[idx], v.reshape(count, -1), TOL["bf16"], "v")


@pytest.mark.parametrize("cap", [1000, NO_SUMS_CAP, 4200])
@pytest.mark.parametrize("count", [0, 1, 127, 128, 129, 256, 257, 330, 384, 385, 640])
def test_count_far_below_capacity(layer, count, cap):
    print("planned gemm", count, cap, flush=True)
    lay, w = layer
    _check(lay, w, SHAPE, 3, 1400, count, cap)


@pytest.mark.parametrize("case", range(len(REGIMES)))
def test_plan_regimes(case):
    shape, count, cap, _ = REGIMES[case]
    print("plan regime", case, count, cap, flush=True)
    B, L = (3, 1400) if cap > 2200 else (2, 1100)
    lay = Layer.from_shape(shape, B, L)
    w = rand_weights(shape, 56, bias=True)
    lay.set_weights(w)
    _check(lay, w, shape, B, L, count, cap)
    lay.close()


# the same in a list with room for half of the tokens at most, whose q|k|v the GEMM may finish (test_gemm_plan_host.py)
HALF = [c for c, (shape, _, cap, _) in enumerate(REGIMES) if cap <= 2100 and shape.hidden == 4096]


@pytest.mark.parametrize("case", HALF)
def test_plan_regimes_of_a_list_of_half_the_tokens(case):
    shape, count, cap, _ = REGIMES[case]
    print("plan regime, half", case, count, cap, flush=True)
    B, L = 4, (cap + 1) // 2
    lay = Layer.from_shape(shape, B, L)
    w = rand_weights(shape, 56, bias=True)
    lay.set_weights(w)
    _check(lay, w, shape, B, L, count, cap)
    lay.close()
