"""Sparse steps over lists whose capacity is far above their count, with more sequences than a wave has lanes, empty
sequences among them, and counts around the 64 entries of a workgroup of the cosine test.  The new contexts against
float32 attention over the caches that the step left, the cosines against 64 bits over the stored contexts, the
selected tokens and offsets exactly by those cosines.

Bounds: contexts at the bf16 bar of every other test; a cosine is three fp32 sums of 4096 products, whose roundings of 2^-24
add up like sqrt(4096): 4e-6, five times that are allowed."""
import numpy as np
import pytest
import torch

from oracle import dyllm_oracle as O
from paper_2603_08026_amd import binding as Bd
from paper_2603_08026_amd.layer import Layer, to_host
from synth import workload as W
from tests.helpers import TOL, assert_close, rand_rows, rand_weights

pytestmark = pytest.mark.gpu

SHAPE = W.LayerShape(hidden=256, n_heads=32, n_kv_heads=32, head_dim=128, ffn=384, dtype="bf16", rope_theta=10000.0)
GROUPED = W.LayerShape(hidden=256, n_heads=32, n_kv_heads=8, head_dim=128, ffn=384, dtype="bf16", rope_theta=10000.0)


def _counts(B, L, n):
    """n entries over B sequences, every third of them empty."""
    live = [b for b in range(B) if b % 3 != 1]
    per = [0] * B
    for i in range(n):
        per[live[i % len(live)]] += 1
    assert max(per) <= L
    return per


@pytest.mark.parametrize("shape,B,L", [(SHAPE, 70, 33), (GROUPED, 70, 33), (SHAPE, 6, 200)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 500])
@pytest.mark.parametrize("full_cap", [False, True])
def test_step(shape, B, L, n, full_cap):
    print("listed step", shape.n_kv_heads, B, L, n, full_cap, flush=True)
    T, s = B * L, shape
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(rand_weights(s, 95, std=0.08))
    gen = torch.Generator().manual_seed(96)
    x0 = torch.randn(B, L, s.hidden, generator=gen)
    idx, off = rand_rows(97, B, L, _counts(B, L, n))
    x1 = x0.clone().view(T, -1)
    x1[idx] += torch.randn(n, s.hidden, generator=gen) * torch.linspace(0.01, 2.0, n)[torch.randperm(n, generator=gen)][:, None]
    lay.full_step(x0.to(torch.bfloat16).cuda())
    old = lay.c.view(T, -1).clone()
    rows = lay.make_list(idx, off, cap=T if full_cap else n)
    tau = 0.9
    out = lay.layer_step(x1.view(B, L, -1).to(torch.bfloat16).cuda(), rows, tau, Bd.IndexList.empty(T, B))
    assert lay.ctx.poll_status() == 0
    got_idx, got_off = lay.read_list(out)
    at = torch.from_numpy(idx.astype(np.int64)).cuda()
    new = lay.c.view(T, -1)
    cos64 = torch.nn.functional.cosine_similarity(new[at].double(), old[at].double(), dim=-1)
    cos = lay.cos[:n]
    assert float((cos.double() - cos64).abs().max()) < 2e-5
    want = idx[cos.cpu().numpy() < np.float32(tau)]
    assert np.array_equal(got_idx, want)
    assert np.array_equal(got_off, np.searchsorted(want, np.arange(B + 1) * L))
    untouched = torch.ones(T, dtype=torch.bool, device="cuda")
    untouched[at] = False
    assert torch.equal(new[untouched], old[untouched])
    # contexts of the listed rows
    q = torch.zeros(rows.cap, s.dq, dtype=torch.bfloat16, device="cuda")
    lay.ctx.qkv_refresh(lay.w, x1.view(B, L, -1).to(torch.bfloat16).cuda(), rows, B, L, lay.cache, q)
    k = lay.k.view(B, L, s.n_kv_heads, s.head_dim).float().cpu()
    v = lay.v.view(B, L, s.n_kv_heads, s.head_dim).float().cpu()
    g = s.n_heads // s.n_kv_heads
    ref = torch.empty(n, s.n_heads, s.head_dim)
    for j in range(n):
        b = int(idx[j]) // L
        qj = q[j].float().cpu().view(s.n_kv_heads, g, s.head_dim)
        p = torch.softmax(torch.einsum("hgd,lhd->hgl", qj, k[b]) / s.head_dim ** 0.5, -1)
        ref[j] = torch.einsum("hgl,lhd->hgd", p, v[b]).reshape(s.n_heads, s.head_dim)
    err = (new[at].float().cpu() - ref.view(n, -1)).abs().max() / ref.abs().max()
    assert float(err) <= TOL["bf16"]
    lay.close()


# Rows that the attention kernel commits (one key split), in 64-row tiles where the list is full and in 128-row tiles where it has room for every
# token: rows per sequence that leave a wave partly filled, waves without a query and a second tile.
COMMITTED = {"heads": (SHAPE, 200, [1, 33, 65, 100, 0, 129]), "groups": (GROUPED, 70, [1, 9, 17, 33, 0] * 4)}


@pytest.mark.parametrize("name", COMMITTED)
@pytest.mark.parametrize("full_cap", [False, True])
@pytest.mark.parametrize("keep_lse", [False, True])
def test_committed_rows(name, full_cap, keep_lse):
    """Contexts, cosines and log-normalisers of the listed rows, and every bit of the others.  A normaliser is the logarithm of a sum of positive
    terms that were each rounded once to the 8 bits of bf16, by 2^-8 of the term at most (half of the spacing above a power of two): the sum
    is off by 2^-8 of itself at most, its logarithm by -log(1 - 2^-8) < 2^-8 + 2^-16; scores and the logarithm in fp32, of values up to 10: 2e-5."""
    print("committed rows", name, full_cap, keep_lse, flush=True)
    s, L, counts = COMMITTED[name]
    B = len(counts)
    T, n = B * L, sum(counts)
    lay = Layer.from_shape(s, B, L, keep_lse=keep_lse)
    lay.set_weights(rand_weights(s, 98, std=0.08))
    gen = torch.Generator().manual_seed(99)
    x = torch.randn(B, L, s.hidden, generator=gen).to(torch.bfloat16).cuda()
    for t in (lay.k, lay.v, lay.c, lay.out) + ((lay.lse,) if keep_lse else ()):
        t.copy_(torch.randn(t.shape, generator=gen).to(t.dtype))
    old = [t.clone() for t in (lay.c.view(T, -1), lay.lse.view(T, -1) if keep_lse else lay.c.view(T, -1))]
    idx, off = rand_rows(100, B, L, counts)
    rows = lay.make_list(idx, off, cap=T if full_cap else n)
    out = lay.layer_step(x, rows, 0.5, Bd.IndexList.empty(T, B))
    assert lay.ctx.poll_status() == 0
    c, cos = lay.c.view(T, -1).clone(), lay.cos[:n].clone()
    lse = lay.lse.view(T, -1).clone() if keep_lse else None
    q = torch.zeros(rows.cap, s.dq, dtype=torch.bfloat16, device="cuda")
    lay.ctx.qkv_refresh(lay.w, x, rows, B, L, lay.cache, q)
    qh, kh, vh = to_host(q)[:n].reshape(n, s.n_heads, s.head_dim), to_host(lay.k), to_host(lay.v)
    at = torch.from_numpy(idx.astype(np.int64)).cuda()
    assert_close(to_host(c)[idx], O.partial_attention(qh, kh, vh, idx, B, L), TOL["bf16"], "contexts")
    cos64 = torch.nn.functional.cosine_similarity(c[at].double(), old[0][at].double(), dim=-1)
    assert float((cos.double() - cos64).abs().max()) < 2e-5
    assert np.array_equal(lay.read_list(out)[0], idx[cos.cpu().numpy() < np.float32(0.5)])
    rest = torch.ones(T, dtype=torch.bool, device="cuda")
    rest[at] = False
    assert torch.equal(c[rest], old[0][rest])
    if keep_lse:
        assert np.abs(lse.cpu().numpy()[idx] - O.partial_lse(qh, kh, idx, B, L)).max() <= 2.0 ** -8 + 2.0 ** -16 + 2e-5
        assert torch.equal(lse[rest], old[1][rest])
    lay.close()
