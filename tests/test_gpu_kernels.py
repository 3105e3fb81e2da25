"""GPU-vs-oracle parity of each boundary call, through the C ABI, on seeded inputs that span
several tiles with ragged tails, empty sequences and the degenerate cases."""
import numpy as np
import pytest
import torch

from oracle import dyllm_oracle as O
from paper_2603_08026_amd import binding as Bd
from paper_2603_08026_amd.layer import Layer, to_device, to_host
from synth import workload as W
from tests.helpers import (TOL, assert_close, assert_index_sets_match, oracle_cfg, rand_rows, rand_weights,
                           small_shape)

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[case]", *a, flush=True)


def _vals(seed, shape, dtype, scale=1.0, *key):
    x = W.philox(seed, "vals", *key).standard_normal(shape, dtype=np.float32) * np.float32(scale)
    return W.round_bf16(x) if dtype == "bf16" else x


# ------------------------------------------------------------------ saliency

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_saliency_candidates_and_commit(dtype):
    _say("saliency candidates", dtype)
    s = small_shape(dtype)
    B, L = 3, 50
    lay = Layer.from_shape(s, B, L)
    D = s.dq
    cache = _vals(1, (B * L, D), dtype)
    idx, off = rand_rows(2, B, L, [17, 0, 33])
    M = idx.size
    # candidates: some identical to the cache, some scaled, some slightly / strongly perturbed, one zero row
    sig = 10.0 ** W.philox(3, "sig").uniform(-4, 0, M)
    new = W.perturbed_rows(cache[idx], sig, 4)
    new[0] = cache[idx[0]]
    new[1] = 2.0 * cache[idx[1]]
    new[2] = 0.0
    cache[idx[3]] = 0.0
    new = W.round_bf16(new) if dtype == "bf16" else new
    tau = 0.99
    ref_cache = cache.astype(np.float64)
    cos_ref, flag_ref = O.saliency(new, ref_cache, idx, tau, commit=True)

    d_cache = to_device(cache, dtype)
    d_new = to_device(new, dtype)
    rows = lay.make_list(idx, off, cap=M + 5)
    cos = torch.full((M + 5,), 7.0, device="cuda")
    flag = torch.full((M + 5,), 9, dtype=torch.uint8, device="cuda")
    lay.ctx.saliency(d_new, d_cache, rows, B, L, tau, cos, flag, commit=True)
    torch.cuda.synchronize()
    cos_g, flag_g = cos.cpu().numpy(), flag.cpu().numpy()
    assert np.max(np.abs(cos_g[:M] - cos_ref)) < 2e-6
    assert cos_g[0] >= 1 - 1e-6 and flag_g[0] == 0  # unchanged context is never salient
    assert abs(cos_g[1] - 1) < 1e-6  # scale invariance of the metric
    assert cos_g[2] == 0.0 and flag_g[2] == 1 and cos_g[3] == 0.0  # zero rows: s = 0, no NaN
    firm = np.abs(cos_ref - tau) > 1e-3
    assert np.array_equal(flag_g[:M][firm], flag_ref[firm].astype(np.uint8))
    assert np.all(cos_g[M:] == 7.0) and np.all(flag_g[M:] == 9)  # nothing written past the count
    assert np.array_equal(to_host(d_cache), ref_cache)  # commit: rows replaced, others untouched
    lay.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_saliency_all_rows_form(dtype):
    _say("saliency all rows", dtype)
    s = small_shape(dtype)
    B, L = 2, 37
    lay = Layer.from_shape(s, B, L)
    a = _vals(5, (B * L, s.dq), dtype)
    sig = 10.0 ** W.philox(6, "sig").uniform(-4, 0, B * L)
    b = W.perturbed_rows(a, sig, 7)
    b = W.round_bf16(b) if dtype == "bf16" else b
    cos_ref, flag_ref = O.saliency(b, a, None, 0.995)
    cos = torch.zeros(B * L, device="cuda")
    flag = torch.zeros(B * L, dtype=torch.uint8, device="cuda")
    d_a = to_device(a, dtype)
    lay.ctx.saliency(to_device(b, dtype), d_a, None, B, L, 0.995, cos, flag, commit=False)
    torch.cuda.synchronize()
    assert np.max(np.abs(cos.cpu().numpy() - cos_ref)) < 2e-6
    firm = np.abs(cos_ref - 0.995) > 1e-3
    assert np.array_equal(flag.cpu().numpy()[firm], flag_ref[firm].astype(np.uint8))
    assert np.array_equal(to_host(d_a), a.astype(np.float64))
    lay.close()


# ------------------------------------------------------------------ compaction

@pytest.mark.parametrize("case", ["candidates", "identity", "empty", "all", "big"])
def test_compact_bit_exact(case):
    _say("compact", case)
    s = small_shape("f32")
    B, L = (4, 300) if case != "big" else (16, 2048)
    lay = Layer.from_shape(s, B, L)
    g = W.philox(8, "compact", case)
    if case == "identity" or case == "big":
        rows_np, off_np, rows = None, None, None
        n = B * L
    else:
        counts = [123, 0, 300, 1]
        rows_np, off_np = rand_rows(9, B, L, counts)
        n = rows_np.size
        rows = lay.make_list(rows_np, off_np, cap=n + 3)
    p = {"empty": 0.0, "all": 1.0}.get(case, 0.3)
    flag_np = (g.uniform(size=n) < p).astype(np.uint8)
    if case == "big":
        flag_np[: 3 * L] = 0  # three leading sequences without any salient token
    idx_ref, off_ref = O.compact(flag_np, rows_np, B, L)
    out = Bd.IndexList.empty(n, B)
    out.idx.fill_(-1)
    flag = torch.from_numpy(np.concatenate([flag_np, np.ones(3, np.uint8)])).cuda()
    lay.ctx.compact(flag, rows, B, L, out)
    idx_g, off_g = lay.read_list(out)
    assert np.array_equal(off_g, off_ref)
    assert np.array_equal(idx_g, idx_ref)
    assert lay.ctx.poll_status() == 0
    lay.close()


def test_compact_capacity_overflow_is_reported():
    _say("compact overflow")
    s = small_shape("f32")
    B, L = 2, 100
    lay = Layer.from_shape(s, B, L)
    flag_np = np.ones(B * L, np.uint8)
    out = Bd.IndexList.empty(50, B)
    guard = torch.full((60,), -7, dtype=torch.int32, device="cuda")
    out = Bd.IndexList(guard[:50], out.offsets)
    lay.ctx.compact(torch.from_numpy(flag_np).cuda(), None, B, L, out)
    assert lay.ctx.poll_status() == Bd.ERR_CAPACITY
    assert lay.ctx.poll_status() == 0  # cleared by the poll
    idx_g, off_g = lay.read_list(out)
    assert np.array_equal(idx_g, np.arange(50)) and off_g.tolist() == [0, 50, 50]
    assert np.all(guard[50:].cpu().numpy() == -7)
    lay.close()


# ------------------------------------------------------------------ q/k/v refresh

@pytest.mark.parametrize("dtype,gqa,dh,bias,counts", [
    ("f32", False, 64, False, [70, 0, 5]), ("f32", True, 128, True, [70, 0, 5]),
    ("bf16", False, 128, False, [70, 0, 5]), ("bf16", True, 64, True, [70, 0, 5]),
    # few rows: the weight-streaming GEMM leaves out the activation copies of absent row blocks
    ("bf16", False, 128, True, [20, 0, 25]), ("bf16", True, 64, False, [3, 0, 9]),
    # 129 .. 320 rows: the 256-row weight-streaming tile, alone and with a short second row tile
    ("bf16", False, 128, True, [90, 0, 80]), ("bf16", True, 64, False, [90, 88, 90])])
def test_qkv_refresh(dtype, gqa, dh, bias, counts):
    _say("qkv_refresh", dtype, gqa, dh, bias, counts)
    s = small_shape(dtype, gqa, dh)
    cfg = oracle_cfg(s)
    B, L = 3, 90
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 11, bias=bias)
    lay.set_weights(w)
    x = _vals(12, (B, L, s.hidden), dtype)
    idx, off = rand_rows(13, B, L, counts)
    k0, v0 = _vals(14, (B * L, s.dkv), dtype), _vals(15, (B * L, s.dkv), dtype)
    lay.k.copy_(to_device(k0, dtype).view_as(lay.k))
    lay.v.copy_(to_device(v0, dtype).view_as(lay.v))
    rows = lay.make_list(idx, off, cap=idx.size + 2)
    q_out = torch.zeros(idx.size + 2, s.dq, dtype=lay.k.dtype, device="cuda")
    lay.ctx.qkv_refresh(lay.w, lay.upload(x), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    n = O.rmsnorm(x.reshape(B * L, -1)[idx], w["g_attn"], cfg.rms_eps)
    q, k, v = O.project_qkv(n, idx % L, w, cfg)
    tol = TOL[dtype]
    assert_close(to_host(q_out)[:idx.size], q.reshape(idx.size, -1), tol, "q")
    kg, vg = to_host(lay.k).reshape(B * L, -1), to_host(lay.v).reshape(B * L, -1)
    assert_close(kg[idx], k.reshape(idx.size, -1), tol, "k rows")
    assert_close(vg[idx], v.reshape(idx.size, -1), tol, "v rows")
    others = np.setdiff1d(np.arange(B * L), idx)
    assert np.array_equal(kg[others], k0[others].astype(np.float64))  # K/V merge leaves the rest alone
    assert np.array_equal(vg[others], v0[others].astype(np.float64))
    assert np.all(to_host(q_out)[idx.size:] == 0)
    lay.close()


# ------------------------------------------------------------------ partial attention

@pytest.mark.parametrize("dtype,gqa,dh,B,L,counts", [
    ("f32", False, 64, 3, 70, [33, 0, 70]),
    ("f32", True, 128, 2, 45, [1, 20]),
    ("bf16", False, 128, 3, 200, [100, 0, 7]),
    ("bf16", True, 64, 2, 333, [65, 129]),
    ("bf16", False, 128, 1, 1024, [106]),
    ("bf16", True, 128, 1, 77, [77]),
    ("bf16", True, 128, 3, 200, [100, 0, 37]),   # grouped heads folded into ragged tiles, an empty sequence
    ("bf16", True, 128, 2, 1100, [19, 150]),     # the same over several key splits of many tiles
])
def test_partial_attention(dtype, gqa, dh, B, L, counts):
    _say("partial_attention", dtype, gqa, dh, B, L, counts)
    s = small_shape(dtype, gqa, dh)
    lay = Layer.from_shape(s, B, L)
    idx, off = rand_rows(21, B, L, counts)
    M = idx.size
    q = _vals(22, (M, s.n_heads, dh), dtype, 1.5)
    k = _vals(23, (B, L, s.n_kv_heads, dh), dtype, 1.5)
    v = _vals(24, (B, L, s.n_kv_heads, dh), dtype)
    ref = O.partial_attention(q, k, v, idx, B, L)
    cap = min(M + 3, B * L)
    rows = lay.make_list(idx, off, cap=cap)
    out = torch.zeros(M + 3, s.dq, dtype=lay.k.dtype, device="cuda")
    qd = torch.zeros(M + 3, s.n_heads, dh, dtype=lay.k.dtype, device="cuda")
    qd[:M] = to_device(q, dtype)
    lay.ctx.partial_attention(qd, to_device(k, dtype), to_device(v, dtype), rows, B, L, out)
    torch.cuda.synchronize()
    assert_close(to_host(out)[:M], ref, TOL[dtype], "context rows")
    assert np.all(to_host(out)[M:] == 0)
    lay.close()


@pytest.mark.parametrize("B,L,counts", [(1, 1100, [150]), (2, 300, [130, 40])])
def test_partial_attention_with_a_moving_softmax_reference(B, L, counts):
    """Keys grow along the sequence, so the largest score of a key tile keeps exceeding the running
    reference of the online softmax by more than the kernel's lazy threshold: the accumulator and
    the pending product of the previous tile are rescaled in the middle of the key sweep, over
    full tiles, a ragged last tile, query tiles with idle waves and several key splits."""
    _say("partial_attention, growing keys", B, L, counts)
    dtype, dh = "bf16", 128
    s = small_shape(dtype, False, dh)
    lay = Layer.from_shape(s, B, L)
    idx, off = rand_rows(31, B, L, counts)
    M = idx.size
    q = _vals(32, (M, s.n_heads, dh), dtype, 1.5)
    ramp = (1.0 + 5.0 * np.arange(L, dtype=np.float32) / L).reshape(1, L, 1, 1)
    k = W.round_bf16(_vals(33, (B, L, s.n_kv_heads, dh), "f32", 1.5) * ramp)
    v = _vals(34, (B, L, s.n_kv_heads, dh), dtype)
    ref = O.partial_attention(q, k, v, idx, B, L)
    rows = lay.make_list(idx, off, cap=M)
    out = torch.zeros(M, s.dq, dtype=lay.k.dtype, device="cuda")
    lay.ctx.partial_attention(to_device(q, dtype), to_device(k, dtype), to_device(v, dtype), rows, B, L, out)
    torch.cuda.synchronize()
    assert_close(to_host(out), ref, TOL[dtype], "context rows")
    lay.close()


def test_partial_attention_special_cases():
    _say("partial_attention special cases")
    s = small_shape("f32")
    B, L = 1, 40
    lay = Layer.from_shape(s, B, L)
    idx, off = np.arange(0, 40, 3, dtype=np.int32), np.array([0, 14], np.int32)
    q = _vals(25, (14, s.n_heads, 64), "f32")
    krow = _vals(26, (1, 1, s.n_kv_heads, 64), "f32")
    k = np.tile(krow, (1, L, 1, 1))  # all keys equal: uniform weights, context = mean of V
    v = _vals(27, (B, L, s.n_kv_heads, 64), "f32")
    out = torch.zeros(14, s.dq, device="cuda")
    lay.ctx.partial_attention(to_device(q, "f32"), to_device(k, "f32"), to_device(v, "f32"),
                              lay.make_list(idx, off), B, L, out)
    want = np.tile(v[0].mean(axis=0).reshape(1, -1), (14, 1))
    assert_close(to_host(out), want, 1e-5, "uniform attention")
    lay.close()
    # a single key: the context is that value row
    lay = Layer.from_shape(s, 2, 1)
    v1 = _vals(28, (2, 1, s.n_kv_heads, 64), "f32")
    out = torch.zeros(2, s.dq, device="cuda")
    lay.ctx.partial_attention(to_device(q[:2], "f32"), to_device(_vals(29, (2, 1, s.n_kv_heads, 64), "f32"), "f32"),
                              to_device(v1, "f32"), lay.make_list(np.array([0, 1], np.int32), np.array([0, 1, 2], np.int32)),
                              2, 1, out)
    assert_close(to_host(out), v1.reshape(2, -1), 1e-6, "single key")
    lay.close()


# ------------------------------------------------------------------ salient FFN

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_salient_ffn(dtype):
    _say("salient_ffn", dtype)
    s = small_shape(dtype)
    cfg = oracle_cfg(s)
    B, L = 2, 150
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 31)
    lay.set_weights(w)
    x = _vals(32, (B * L, s.hidden), dtype)
    c = _vals(33, (B * L, s.dq), dtype)
    out0 = _vals(34, (B * L, s.hidden), dtype)
    idx, off = rand_rows(35, B, L, [101, 9])
    ref = out0.astype(np.float64)
    O.salient_ffn(x, c, idx, w, cfg, ref)
    d_out = to_device(out0, dtype)
    lay.ctx.salient_ffn(lay.w, to_device(x, dtype), to_device(c, dtype), lay.make_list(idx, off, cap=idx.size + 1),
                        B, L, d_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    assert_close(got[idx], ref[idx], TOL[dtype], "ffn rows")
    others = np.setdiff1d(np.arange(B * L), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    lay.close()


@pytest.mark.parametrize("M,cap", [(520, 520), (520, 820), (700, 701), (1024, 1024), (397, 900), (769, 1600)])
def test_large_tile_regime_with_ragged_row_counts(M, cap):
    """More than 320 list entries: 256-row GEMM tiles.  A last row tile with few rows runs the
    shortened loop and is numbered after the full tiles on every XCD; a list shorter than its capacity
    moves that split away from what the host sized the grid for."""
    _say("large tiles, ragged", M, cap)
    dtype = "bf16"
    s = small_shape(dtype)
    cfg = oracle_cfg(s)
    B, L = 4, 400
    T = B * L
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 141, bias=True)
    lay.set_weights(w)
    per = [M // B + (1 if b < M % B else 0) for b in range(B)]
    idx, off = rand_rows(142, B, L, per)
    rows = lay.make_list(idx, off, cap=cap)
    tol = TOL[dtype]
    # q/k/v refresh (raw GEMM + row kernel)
    x = _vals(143, (B, L, s.hidden), dtype)
    q_out = torch.zeros(cap, s.dq, dtype=lay.k.dtype, device="cuda")
    lay.ctx.qkv_refresh(lay.w, lay.upload(x), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    n = O.rmsnorm(x.reshape(T, -1)[idx], w["g_attn"], cfg.rms_eps)
    q, k, v = O.project_qkv(n, idx % L, w, cfg)
    assert_close(to_host(q_out)[:M], q.reshape(M, -1), tol, "q")
    assert_close(to_host(lay.k).reshape(T, -1)[idx], k.reshape(M, -1), tol, "k rows")
    assert_close(to_host(lay.v).reshape(T, -1)[idx], v.reshape(M, -1), tol, "v rows")
    assert np.all(to_host(q_out)[M:] == 0)
    # out-projection + FFN (raw GEMM, fused SwiGLU and residual epilogues)
    c = _vals(144, (T, s.dq), dtype)
    out0 = _vals(145, (T, s.hidden), dtype)
    ref = out0.astype(np.float64)
    O.salient_ffn(x.reshape(T, -1), c, idx, w, cfg, ref)
    d_out = to_device(out0, dtype)
    lay.ctx.salient_ffn(lay.w, lay.upload(x), to_device(c, dtype), rows, B, L, d_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    assert_close(got[idx], ref[idx], tol, "ffn rows")
    others = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    lay.close()


@pytest.mark.parametrize("hidden,heads,kv_heads,ffn", [(512, 6, 1, 512), (256, 4, 4, 512), (384, 6, 6, 256)])
def test_four_wave_256x256_tiles_with_short_k_and_stacked_weights(hidden, heads, kv_heads, ffn):
    """Enough rows that the planner takes the 256 x 256 tiles at small widths (more than 256 tiles, so
    every workgroup walks several of them and refills its LDS ring for the next): K of 8, 4 and 6
    slices (4 is the shortest a bf16 configuration can have), a column tile that spans the q, k and v matrices (q|k|v is 384 + 64 + 64 columns in the
    first case), and a last row tile of 156 rows (one wave pair multiplies four 32-row blocks, the
    other one)."""
    _say("256x256 tiles, short K", hidden, heads, kv_heads, ffn)
    dtype = "bf16"
    s = W.LayerShape(hidden=hidden, n_heads=heads, n_kv_heads=kv_heads, head_dim=64, ffn=ffn, dtype=dtype,
                     rope_theta=10000.0)
    cfg = oracle_cfg(s)
    B, L = 20, 2048
    T = B * L
    M = T - 100
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 151, bias=True)
    lay.set_weights(w)
    per = [M // B + (1 if b < M % B else 0) for b in range(B)]
    idx, off = rand_rows(152, B, L, per)
    rows = lay.make_list(idx, off, cap=T)
    tol = TOL[dtype]
    x = _vals(153, (B, L, s.hidden), dtype)
    q_out = torch.zeros(T, s.dq, dtype=lay.k.dtype, device="cuda")
    lay.ctx.qkv_refresh(lay.w, lay.upload(x), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    n = O.rmsnorm(x.reshape(T, -1)[idx], w["g_attn"], cfg.rms_eps)
    q, k, v = O.project_qkv(n, idx % L, w, cfg)
    assert_close(to_host(q_out)[:M], q.reshape(M, -1), tol, "q")
    assert_close(to_host(lay.k).reshape(T, -1)[idx], k.reshape(M, -1), tol, "k rows")
    assert_close(to_host(lay.v).reshape(T, -1)[idx], v.reshape(M, -1), tol, "v rows")
    c = _vals(154, (T, s.dq), dtype)
    out0 = _vals(155, (T, s.hidden), dtype)
    ref = out0.astype(np.float64)
    O.salient_ffn(x.reshape(T, -1), c, idx, w, cfg, ref)
    d_out = to_device(out0, dtype)
    lay.ctx.salient_ffn(lay.w, lay.upload(x), to_device(c, dtype), rows, B, L, d_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    assert_close(got[idx], ref[idx], tol, "ffn rows")
    others = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    lay.close()


@pytest.mark.parametrize("M,cap,ffn", [(2075, 2075, 4096), (2060, 2075, 4096), (1990, 2075, 4096), (1819, 1819, 12288),
                                       (1800, 1819, 12288)])
def test_short_last_row_tile_streamed_in_a_launch_of_its_own(M, cap, ffn):
    """Widths at which eight full 256-row tiles fill the chip's 256 CUs exactly (q|k|v 8192, out-projection
    and gate|up 4096 columns over K = 4096), so that the 27 rows of a ninth row tile would open a round of their own:
    rows 2048.. go to the weight-streaming tiles, whose K split (2 for q|k|v, 4 for the out-projection) differs from the
    row tiles' (none).  With fewer rows than the capacity there are fewer streamed rows (2060) or none and a partial row
    tile (1990).  The down projection's plans for these counts stream nothing: without a K split at 4096 FFN columns,
    split in two at 12288 (1819 and 1800 rows, where the other GEMMs stream nothing either).  The plans are checked in
    test_gemm_plan_host.py; streamed rows of the down projection are in test_gpu_planned_gemm.py."""
    _say("streamed last row tile", M, cap)
    dtype = "bf16"
    s = W.LayerShape(hidden=4096, n_heads=32, n_kv_heads=16, head_dim=128, ffn=ffn, dtype=dtype, rope_theta=10000.0)
    cfg = oracle_cfg(s)
    B, L = 2, 1100
    T = B * L
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 171, bias=True)
    lay.set_weights(w)
    per = [M // B + (1 if b < M % B else 0) for b in range(B)]
    idx, off = rand_rows(172, B, L, per)
    rows = lay.make_list(idx, off, cap=cap)
    tol = TOL[dtype]
    x = _vals(173, (B, L, s.hidden), dtype)
    q_out = torch.zeros(cap, s.dq, dtype=lay.k.dtype, device="cuda")
    lay.ctx.qkv_refresh(lay.w, lay.upload(x), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    n = O.rmsnorm(x.reshape(T, -1)[idx], w["g_attn"], cfg.rms_eps)
    q, k, v = O.project_qkv(n, idx % L, w, cfg)
    assert_close(to_host(q_out)[:M], q.reshape(M, -1), tol, "q")
    assert_close(to_host(lay.k).reshape(T, -1)[idx], k.reshape(M, -1), tol, "k rows")
    assert_close(to_host(lay.v).reshape(T, -1)[idx], v.reshape(M, -1), tol, "v rows")
    assert np.all(to_host(q_out)[M:] == 0)
    c = _vals(174, (T, s.dq), dtype)
    out0 = _vals(175, (T, s.hidden), dtype)
    ref = out0.astype(np.float64)
    O.salient_ffn(x.reshape(T, -1), c, idx, w, cfg, ref)
    d_out = to_device(out0, dtype)
    lay.ctx.salient_ffn(lay.w, lay.upload(x), to_device(c, dtype), rows, B, L, d_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    assert_close(got[idx], ref[idx], tol, "ffn rows")
    others = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    lay.close()


@pytest.mark.parametrize("B,L,M,cap,bias", [(16, 2048, 32668, 32768, True), (16, 1100, 16411, 16411, True),
                                              (16, 1100, 16400, 16411, False), (16, 1100, 9000, 16411, True)])
def test_qkv_refresh_with_128_wide_heads_at_many_rows(B, L, M, cap, bias):
    """bf16 with 128-wide heads and many rows (grouped-query shape: 4 query heads, 2 key/value heads, so a column tile
    holds q heads, or a k and a v head pair), with and without biases.  Cases: a last row tile of 156 rows beside full
    256 x 128 tiles; 16384 + 27 rows, where the 27 go to the weight-streaming tiles behind 256 x 256 ones; fewer rows than
    the capacity, so that 16 rows are streamed, or none and the last row tile is a partial one.  Rows outside the list
    keep their cached keys and values bit for bit.  The plans are checked in test_gemm_plan_host.py."""
    _say("q/k/v refresh, 128-wide heads, many rows", B, L, M, cap)
    dtype = "bf16"
    s = W.LayerShape(hidden=1024, n_heads=4, n_kv_heads=2, head_dim=128, ffn=512, dtype=dtype, rope_theta=10000.0)
    cfg = oracle_cfg(s)
    T = B * L
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 181, bias=bias)
    lay.set_weights(w)
    per = [M // B + (1 if b < M % B else 0) for b in range(B)]
    idx, off = rand_rows(182, B, L, per)
    rows = lay.make_list(idx, off, cap=cap)
    tol = TOL[dtype]
    x = _vals(183, (B, L, s.hidden), dtype)
    k0, v0 = to_host(lay.k).reshape(T, -1).copy(), to_host(lay.v).reshape(T, -1).copy()
    q_out = torch.zeros(cap, s.dq, dtype=lay.k.dtype, device="cuda")
    lay.ctx.qkv_refresh(lay.w, lay.upload(x), rows, B, L, lay.cache, q_out)
    torch.cuda.synchronize()
    n = O.rmsnorm(x.reshape(T, -1)[idx], w["g_attn"], cfg.rms_eps)
    q, k, v = O.project_qkv(n, idx % L, w, cfg)
    assert_close(to_host(q_out)[:M], q.reshape(M, -1), tol, "q")
    k1, v1 = to_host(lay.k).reshape(T, -1), to_host(lay.v).reshape(T, -1)
    assert_close(k1[idx], k.reshape(M, -1), tol, "k rows")
    assert_close(v1[idx], v.reshape(M, -1), tol, "v rows")
    assert np.all(to_host(q_out)[M:] == 0)
    others = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(k1[others], k0[others]) and np.array_equal(v1[others], v0[others])
    lay.close()


def test_eight_wave_fallback_of_the_large_tile_regime():
    """Gathered operands of 4 GiB or more cannot be addressed by the four-wave loop's 32-bit lane
    offsets and take the eight-wave 256 x 128 kernels; the library's diagnostic switch sends every
    call there, and the ragged large-tile cases must still agree with the oracle."""
    import os
    os.environ["DYLLM_GEMM_NO_RING"] = "1"
    try:
        test_large_tile_regime_with_ragged_row_counts(700, 701)
        test_large_tile_regime_with_ragged_row_counts(769, 1600)
    finally:
        del os.environ["DYLLM_GEMM_NO_RING"]


def test_error_paths_do_not_launch():
    _say("error paths")
    s = small_shape("f32")
    lay = Layer.from_shape(s, 2, 32, max_rows=16)
    lay.set_weights(rand_weights(s, 36))
    x = lay.upload(_vals(37, (2, 32, s.hidden), "f32"))
    big = Bd.IndexList.empty(17, 2)
    with pytest.raises(Bd.DyllmError) as e:
        lay.layer_step(x, big, 0.99)
    assert e.value.code == Bd.ERR_CAPACITY
    with pytest.raises(Bd.DyllmError) as e:
        lay.full_step(x)  # needs max_rows >= B*L
    assert e.value.code == Bd.ERR_CAPACITY
    with pytest.raises(Bd.DyllmError) as e:
        lay.ctx.layer_step(lay.w, lay.cache, lay.out, Bd.IndexList.empty(4, 2), 2, 32, 0.99, lay.idx_out, None)
    assert e.value.code == -1  # x aliases the output cache
    with pytest.raises(Bd.DyllmError) as e:
        lay.ctx.full_step(lay.w, lay.cache, x, 3, 32)
    assert e.value.code == -2
    torch.cuda.synchronize()
    lay.close()


@pytest.mark.parametrize("ffn,rows", [(640, [70, 40]), (384, [101, 9]), (1024, [5, 0]), (384, [30, 20]), (640, [33, 31]),
                                      # 129 .. 320 rows: one 256-row tile, and a short second one
                                      (640, [150, 100]), (384, [129, 0]), (1024, [200, 119]), (384, [256, 1])])
def test_salient_ffn_weight_streaming_tiles(ffn, rows):
    """bf16, at most 320 rows: gate|up tiles hold 48 + 48 (F a multiple of 48) or 64 + 64 columns and
    SwiGLU is applied inside the GEMM; the widths here reach both forms and several column tiles, the
    row counts the 128-row and the 256-row tile."""
    _say("salient_ffn streaming tiles", ffn, rows)
    s = W.LayerShape(hidden=256, n_heads=4, n_kv_heads=4, head_dim=64, ffn=ffn, dtype="bf16", rope_theta=10000.0)
    cfg = oracle_cfg(s)
    B, L = 2, max(150, max(rows) + 4)
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 61)
    lay.set_weights(w)
    x = _vals(62, (B * L, s.hidden), "bf16")
    c = _vals(63, (B * L, s.dq), "bf16")
    out0 = _vals(64, (B * L, s.hidden), "bf16")
    idx, off = rand_rows(65, B, L, rows)
    ref = out0.astype(np.float64)
    O.salient_ffn(x, c, idx, w, cfg, ref)
    d_out = to_device(out0, "bf16")
    lay.ctx.salient_ffn(lay.w, to_device(x, "bf16"), to_device(c, "bf16"), lay.make_list(idx, off, cap=idx.size + 1),
                        B, L, d_out)
    torch.cuda.synchronize()
    got = to_host(d_out)
    assert_close(got[idx], ref[idx], TOL["bf16"], "ffn rows")
    others = np.setdiff1d(np.arange(B * L), idx)
    assert np.array_equal(got[others], out0[others].astype(np.float64))
    lay.close()


# ------------------------------------------------------------------ weight re-layout

@pytest.mark.parametrize("n_out,n_in", [(32, 64), (96, 192), (4096 + 512, 4096), (384, 12288)])
def test_pack_weight_bit_exact(n_out, n_in):
    """dyllm_pack_weight against the layout its declaration states, written as a numpy re-shape:
    panels of 32 rows, slices of 64 columns, slice-major inside a panel."""
    _say("pack weight", n_out, n_in)
    bits = W.philox(41, "packbits", n_out, n_in).integers(0, 1 << 16, size=(n_out, n_in), dtype=np.uint16)
    src = torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
    dst = torch.full_like(src, float("nan"))
    Bd.pack_weight(src, dst)
    torch.cuda.synchronize()
    got = dst.view(torch.int16).cpu().numpy().view(np.uint16).ravel()
    want = bits.reshape(n_out // 32, 32, n_in // 64, 64).transpose(0, 2, 1, 3).ravel()
    assert np.array_equal(got, want)
    # one element by the stated formula
    n, k = n_out - 3, n_in - 5
    assert got[((n // 32) * (n_in // 64) + k // 64) * 2048 + (n % 32) * 64 + k % 64] == bits[n, k]


def test_pack_weight_rejects_bad_sizes():
    _say("pack weight errors")
    a = torch.zeros(48, 64, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(Bd.DyllmError) as e:
        Bd.pack_weight(a, torch.empty_like(a))  # 48 rows: not a multiple of 32
    assert e.value.code == -3
    b = torch.zeros(32, 96, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(Bd.DyllmError) as e:
        Bd.pack_weight(b, torch.empty_like(b))  # 96 columns: not a multiple of 64
    assert e.value.code == -3
    c = torch.zeros(32, 64, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(Bd.DyllmError) as e:
        Bd.pack_weight(c, c)  # in place
    assert e.value.code == -1
