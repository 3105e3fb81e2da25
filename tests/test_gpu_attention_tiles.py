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


# bf16, 64-row tiles: two wave columns share the keys of a tile of 64 and their sums are merged as fma(other, c1, own * c0), the
# first column's product rounded.  Scores are equal within a column, so that every weight is 1 and the columns' sums are whole
# numbers A and -S; c1 is 1 and S the whole part of A c0, so that what is left is what the rounding of A c0 decides: in units
# of the row sum, fl(A c0) - S against fl(A c0 - S) differ by up to 1/16.  c0 = 2^d is taken from the neighbours of the
# rounded power (the hardware's has an error of one unit).
def test_merge_of_wave_columns_rounds_the_first_product():
    s = W.LayerShape(hidden=128, n_heads=1, n_kv_heads=1, head_dim=128, ffn=128, dtype="bf16")
    f32 = np.float32
    sc = np.uint32(0x3e0293ee).view(f32)  # log2(e) / sqrt(128)
    q0, k0, k1 = 8.0, -2.0, 1.5
    d = f32(f32(q0 * k0) * sc) - f32(f32(q0 * k1) * sc)
    c0s = [np.exp2(np.float64(d)).astype(f32)]
    c0s = [np.nextafter(c0s[0], f32(0)), c0s[0], np.nextafter(c0s[0], f32(1))]
    rng = np.random.Generator(np.random.Philox(5))
    parts = np.concatenate([rng.integers(128, 256, (1, 128)), rng.integers(0, 256, (2, 128))])
    unit = np.array([[65536.0], [256.0], [1.0]])
    A = (parts * unit).sum(0)
    S = np.floor(A * np.float64(c0s[1]))
    s_parts = np.stack([S // 65536, S // 256 % 256, S % 256])
    v = np.zeros((64, 128))
    v[0:3] = parts * unit
    v[32:35] = -s_parts * unit
    k, q = np.zeros((64, 128)), np.zeros((1, 128))
    k[:32, 0], k[32:, 0], q[0, 0] = k0, k1, q0
    lay = Layer.from_shape(s, 1, 64)
    rows = lay.make_list(np.array([5], np.int32), np.array([0, 1], np.int32))
    out = torch.zeros(1, 128, dtype=torch.bfloat16, device="cuda")
    dev = [torch.tensor(a, dtype=torch.bfloat16, device="cuda") for a in (q, k, v)]
    for a, t in zip((q, k, v), dev):
        assert (t.double().cpu().numpy() == a).all()
    lay.ctx.partial_attention(dev[0], dev[1], dev[2], rows, 1, 64, out)
    got = out.double().cpu().numpy()[0]
    lay.close()

    def miss(c0):  # (largest error, columns that tell the two roundings apart)
        two = (A * np.float64(c0)).astype(f32).astype(np.float64) - S
        one = (A * np.float64(c0) - S).astype(f32).astype(np.float64)
        err = np.abs(got * (32.0 * np.float64(c0) + 32.0) - two)
        return err.max(), int((np.abs(two - one) > 0.03).sum())
    err, telling = min(miss(c) for c in c0s)
    assert telling >= 20 and err < 0.01, (err, telling)  # (bf16 rounds results of at most 2 by 2^-8)


# bf16, head_dim 128: which keys are copied past the L2 is decided by the list's room (64-row tiles) or by each sequence's rows
# (128-row tiles), for keys and values of 64 MiB and more: the lengths of 1409 tokens, the first in 64-row tiles.  Sequences of
# no, one, one full and several query tiles; key counts that leave stages and tiles of the pipeline partly filled.
@pytest.mark.parametrize("heads,kv,L,counts", [(h, kv, L, c) for h, kv in ((4, 4), (8, 2), (64, 32))
                                               for L, c in ((70, [0, 1, 70]), (300, [16, 64, 65]), (600, [128, 0, 300]))]
                         + [(64, 32, 1409, c) for c in ([20, 0, 32], [1, 64, 31], [128, 0, 300], [64, 65, 63])])
def test_copies_past_the_l2(heads, kv, L, counts):
    print("attention past the L2", heads, kv, L, counts, flush=True)
    s = W.LayerShape(hidden=128, n_heads=heads, n_kv_heads=kv, head_dim=128, ffn=128, dtype="bf16")
    B = len(counts)
    g = torch.Generator().manual_seed(L + heads)
    k, v = (torch.randn(B, L, kv * 128, generator=g).bfloat16().cuda() for _ in range(2))
    full = torch.randn(B * L, s.dq, generator=g).bfloat16().cuda()  # a query for every token
    idx, off = rand_rows(73, B, L, counts)
    lay = Layer.from_shape(s, B, L)
    outs = []
    for cap in (idx.size, B * L):
        rows = lay.make_list(idx, off, cap=cap)
        q, out = torch.zeros(cap, s.dq, dtype=torch.bfloat16, device="cuda"), torch.zeros(cap, s.dq, dtype=torch.bfloat16, device="cuda")
        q[:idx.size] = full[torch.from_numpy(idx).long().cuda()]
        lay.ctx.partial_attention(q, k, v, rows, B, L, out)
        outs.append(out[:idx.size].float().cpu().numpy())
    lay.close()
    # (lists of other room may have other tiles and key splits: sums in another order, each rounded to 8 bits once)
    for got in outs:
        ref = O.partial_attention(to_host(full).reshape(B * L, heads, 128)[idx], to_host(k).reshape(B, L, kv, 128), to_host(v).reshape(B, L, kv, 128), idx, B, L)
        assert_close(got, ref.reshape(idx.size, -1), 2e-2, "context rows")


# bf16, head_dim 128, two kernels: 128-row tiles with key tiles of 32 and 64-row tiles with key tiles of 64.  The loop over the key tiles is
# unrolled over four stages from eight tiles on, takes the others but the last four one by one and ends in tiles of their own;
# rows leave 4 * i + sub to an access; a reference that moves takes the half of the pending probabilities along.  So: row
# counts around those of a wave and a tile, keys that grow so that the reference moves in every tile, and for each kernel, with all keys in one
# split (rows finished in place), numbers of key tiles from one to ten and above, the last of them full and not.  Few rows are cut over
# keys as well (2 and 6 heads: partial sums, merged by a kernel of their own).
SWEEP_COUNTS = {1: (1, 3, 31, 33, 64, 65, 0, 127, 129), 4: (1, 8, 16, 17, 0, 32, 33, 35, 16)}  # by heads of a group
SWEEP = ([(h, kv, 1, L) for h, kv in ((2, 2), (6, 2)) for L in (1, 31, 33, 64, 97, 128, 129, 161, 255, 257, 300)]
         + [(16, 16, 1, L) for L in (1, 64, 65, 90, 97, 128, 129, 161, 200, 225, 257, 300, 320, 350, 385, 400, 449, 512, 513, 577, 769)]
         + [(32, 8, 1, L) for L in (40, 200, 257, 449, 513, 577)] + [(16, 16, 4, L) for L in (1, 33, 64)])


def sweep_lists(heads, kv, times, L):
    """The lists of a case: ids, offsets, and the capacities they are given."""
    counts = [min(L, c) for c in (SWEEP_COUNTS.get(heads // kv) or SWEEP_COUNTS[1])] * times
    idx, off = rand_rows(75, len(counts), L, counts)
    return idx, off, (idx.size, len(counts) * L)


# Probabilities and results are rounded to bf16 once each (2^-8 of a weighted mean of values within 5): 2e-2.
@pytest.mark.parametrize("heads,kv,times,L", SWEEP)
@pytest.mark.parametrize("steep", [0.0, 0.3])
def test_bf16_attention_sweep(heads, kv, times, L, steep):
    print("bf16 attention sweep", heads, kv, times, L, steep, flush=True)
    s = W.LayerShape(hidden=128, n_heads=heads, n_kv_heads=kv, head_dim=128, ffn=128, dtype="bf16")
    idx, off, caps = sweep_lists(heads, kv, times, L)
    B = off.size - 1
    g = torch.Generator().manual_seed(17 * L + heads)
    k, v = (torch.randn(B, L, kv, 128, generator=g) for _ in range(2))
    q = torch.randn(B * L, heads, 128, generator=g)
    q[..., 0] = 12.0
    k[..., 0] += steep * torch.arange(L).view(1, L, 1)  # scores rise by 0.3 * 12 / sqrt(128) a key: 15 and 29 powers of two a tile
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    ref = O.partial_attention(q.float().numpy()[idx], k.float().numpy(), v.float().numpy(), idx, B, L)
    lay = Layer.from_shape(s, B, L)
    for cap in caps:
        rows = lay.make_list(idx, off, cap=cap)
        qd = torch.zeros(cap, s.dq, dtype=torch.bfloat16, device="cuda")
        qd[:idx.size] = q.view(B * L, -1)[torch.from_numpy(idx).long()].cuda()
        out = torch.full((cap, s.dq), -7.0, dtype=torch.bfloat16, device="cuda")
        lay.ctx.partial_attention(qd, k.cuda(), v.cuda(), rows, B, L, out)
        torch.cuda.synchronize()
        assert_close(to_host(out)[:idx.size], ref.reshape(idx.size, -1), 2e-2, "context rows")
        assert (out[idx.size:] == -7.0).all()
    lay.close()
