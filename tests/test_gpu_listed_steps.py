"""Sparse steps over lists whose capacity is far above their count, with more sequences than a wave has lanes, empty
sequences among them, and counts around the 64 entries of a workgroup of the cosine test.  The new contexts against
float32 attention over the caches that the step left, the cosines against 64 bits over the stored contexts, the
selected tokens and offsets exactly by those cosines.

Bounds: contexts at the bf16 bar of every other test; a cosine is three fp32 sums of 4096 products, whose roundings of 2^-24
add up like sqrt(4096): 4e-6, five times that are allowed."""
import numpy as np
import pytest
import torch

from paper_2603_08026_amd import binding as Bd
from paper_2603_08026_amd.layer import Layer
from synth import workload as W
from tests.helpers import TOL, rand_rows, rand_weights

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
