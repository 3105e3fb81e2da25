"""fp32 projections that normalise their rows on the way and finish them (q|k|v with bias, rotation and merge; the FFN half with
residual and norm), against the same steps in 64 bits: rows at the edges of 16- and 32-row tiles, one and two 16-column
blocks a tile (few and many tiles), heads of 64 and 128 columns, grouped heads, bias, sequence lengths that are no power of two,
widths with fewer K steps than waves.  fp32 sums of at most 2816 products of order one: 1e-5 of the result's norm."""
import pytest
import torch

from paper_2603_08026_amd import binding as Bd
from synth import workload as W
from tests.helpers import rand_weights

SHAPES = {
    "dh64": W.LayerShape(hidden=256, n_heads=4, n_kv_heads=4, head_dim=64, ffn=768, dtype="f32"),
    "dh64-gqa": W.LayerShape(hidden=320, n_heads=6, n_kv_heads=2, head_dim=64, ffn=448, dtype="f32"),
    "dh128": W.LayerShape(hidden=64, n_heads=6, n_kv_heads=3, head_dim=128, ffn=1536, dtype="f32"),
    # every wave with several steps of K
    "wide": W.LayerShape(hidden=1024, n_heads=16, n_kv_heads=16, head_dim=64, ffn=2816, dtype="f32"),
}


def _norm(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g


@pytest.mark.gpu
@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 300, 777])
@pytest.mark.parametrize("bias", [False, True])
def test_qkv_and_ffn_rows(shape, n, bias):
    from paper_2603_08026_amd.layer import Layer
    s, B, L = SHAPES[shape], 3, 277
    print("fp32 rows", shape, n, bias, flush=True)
    g = torch.Generator().manual_seed(n)
    ids = torch.sort(torch.randperm(B * L, generator=g)[:n])[0]
    off = torch.tensor([int((ids < b * L).sum()) for b in range(B + 1)], dtype=torch.int32).cuda()
    x = torch.randn(B, L, s.hidden, generator=g)
    c = torch.randn(B * L, s.dq, generator=g)
    lay = Layer.from_shape(s, B, L)
    w = rand_weights(s, 81, bias=bias)
    lay.set_weights(w)
    lst = Bd.IndexList(ids.to(torch.int32).cuda(), off)
    q = torch.zeros(n, s.dq, device="cuda")
    lay.k.fill_(5.0)
    lay.v.fill_(-7.0)
    lay.out.fill_(2.0)
    xd = x.cuda()
    lay.ctx.qkv_refresh(lay.w, xd, lst, B, L, lay.cache, q)
    lay.ctx.salient_ffn(lay.w, xd, c.cuda(), lst, B, L, lay.out)
    k, v, out = lay.k.view(B * L, -1).cpu(), lay.v.view(B * L, -1).cpu(), lay.out.view(B * L, -1).cpu()
    lay.close()
    w = {a: torch.as_tensor(b).double() for a, b in w.items() if b is not None}
    rows = x.view(B * L, -1)[ids].double()
    nrm = _norm(rows, w["g_attn"], s.rms_eps)

    def heads(m, b, turn):
        y = nrm @ w[m].t() + (w[b] if bias else 0)
        if not turn:
            return y
        y = y.view(n, -1, s.head_dim)
        half = s.head_dim // 2
        a = ((ids % L).double()[:, None] * s.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64) / s.head_dim))[:, None, :]
        lo, hi = y[..., :half], y[..., half:]
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1).reshape(n, -1)

    def close(got, want, what):
        err = ((got.double() - want).norm() / want.norm()).item()
        assert err <= 1e-5, (what, err)

    close(q.cpu(), heads("wq", "bq", True), "q")
    close(k[ids], heads("wk", "bk", True), "k")
    close(v[ids], heads("wv", "bv", False), "v")
    h = rows + c[ids].double() @ w["wo"].t()
    f = _norm(h, w["g_ffn"], s.rms_eps)
    close(out[ids], h + (torch.nn.functional.silu(f @ w["w_gate"].t()) * (f @ w["w_up"].t())) @ w["w_down"].t(), "out")
    rest = torch.ones(B * L, dtype=torch.bool)
    rest[ids] = False
    assert (k[rest] == 5.0).all() and (v[rest] == -7.0).all() and (out[rest] == 2.0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("result", ["q", "k", "v"])
@pytest.mark.parametrize("n", [17, 300, 777])
def test_results_in_the_place_of_x(result, n):
    """x may be handed over for one of the results: its rows are read before any is written."""
    from paper_2603_08026_amd.layer import Layer
    s, B, L = SHAPES["dh64"], 3, 277
    print("fp32 rows over x", result, n, flush=True)
    g = torch.Generator().manual_seed(n)
    ids = torch.sort(torch.randperm(B * L, generator=g)[:n])[0]
    off = torch.tensor([int((ids < b * L).sum()) for b in range(B + 1)], dtype=torch.int32).cuda()
    lst = Bd.IndexList(ids.to(torch.int32).cuda(), off)
    x = torch.randn(B, L, s.hidden, generator=g).cuda()
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(rand_weights(s, 82, bias=True))
    outs = []
    for shared in (False, True):
        t = {r: torch.full((B * L, s.dq), 3.0, device="cuda") for r in "qkv"}
        xd = x.clone()
        if shared:
            t[result] = xd.view(B * L, -1)
        cache = Bd.LayerCache(t["k"].data_ptr(), t["v"].data_ptr(), lay.c.data_ptr(), lay.out.data_ptr())
        lay.ctx.qkv_refresh(lay.w, xd, lst, B, L, cache, t["q"])
        at = ids.cuda()
        outs.append([t["q"][:n].clone(), t["k"][at].clone(), t["v"][at].clone()])
    lay.close()
    for name, a, b in zip("qkv", *outs):
        assert ((a - b).norm() / a.norm()).item() <= 1e-6, name  # (the norm's factor before the products and after them)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("n", [16, 400])
def test_rows_that_are_not_finite_or_overflow(shape, n):
    """The factor of a row's norm comes after the products: a row of NaN, of one infinity, of values whose squares overflow (the factor
    is 0) and of values whose products would as well, as if each element were normalised first; the other rows keep their bits."""
    from paper_2603_08026_amd.layer import Layer
    s, B, L = SHAPES[shape], 1, 401
    print("fp32 rows, not finite", shape, n, flush=True)
    g = torch.Generator().manual_seed(5)
    x = torch.randn(L, s.hidden, generator=g)
    odd = x.clone()
    odd[1, 3], odd[4, 7], odd[6], odd[8] = float("nan"), float("inf"), 1e20 * torch.sign(x[6]), 3e38 * torch.sign(x[8])
    odd[10] = 3e38
    lst = Bd.IndexList(torch.arange(n, dtype=torch.int32, device="cuda"), torch.tensor([0, n], dtype=torch.int32, device="cuda"))
    lay = Layer.from_shape(s, B, L)
    lay.set_weights(rand_weights(s, 83, std=0.5))
    c = torch.zeros(L, s.dq, device="cuda")  # (the residual rows are x)
    outs = []
    for rows in (x, odd):
        q = torch.zeros(n, s.dq, device="cuda")
        xd = rows.cuda()
        lay.ctx.qkv_refresh(lay.w, xd, lst, B, L, lay.cache, q)
        lay.ctx.salient_ffn(lay.w, xd, c, lst, B, L, lay.out)
        outs.append([t.clone() for t in (q, lay.k.view(L, -1)[:n], lay.v.view(L, -1)[:n], lay.out.view(L, -1)[:n])])
    lay.close()
    same = [r for r in range(n) if r not in (1, 4, 6, 8, 10)]
    for name, a, b in zip(("q", "k", "v", "out"), *outs):
        assert torch.equal(a[same], b[same]), name
        assert torch.isnan(b[[1, 4]]).all(), name
        if name == "out":  # nothing is added to rows whose norm is 0
            assert torch.equal(b[[6, 8, 10]].cpu(), odd[[6, 8, 10]]), name
        else:
            assert (b[[6, 8, 10]] == 0).all(), name
