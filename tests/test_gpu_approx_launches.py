"""The approximate step's launches: the update's attention and the exact rows in one launch against the same two in launches of their
own (a layer that keeps log-normalisers merges its exact rows in another kernel, so they cannot share the launch); candidates
that gather the rows normalised for q against candidates normalised by themselves (a layer step cannot know that a window's
list holds tokens of the window only, the generation loop's step can)."""
import pytest
import torch

from paper_2603_08026_amd import binding as Bd
from paper_2603_08026_amd.layer import Layer, Stack
from synth import workload as W
from tests.helpers import rand_rows, rand_weights

pytestmark = pytest.mark.gpu

CACHES = ("k", "v", "c", "out")


def _inputs(s, B, L, row_lo, counts, seed):
    g = torch.Generator().manual_seed(seed)
    x0 = torch.randn(B, L, s.hidden, generator=g)
    idx, off = rand_rows(seed, B, L - row_lo, counts)
    idx = idx // (L - row_lo) * L + idx % (L - row_lo) + row_lo
    x1 = x0.clone().view(B * L, -1)
    x1[torch.from_numpy(idx).long()] = torch.randn(idx.size, s.hidden, generator=g)
    return x0.bfloat16().cuda(), x1.view(B, L, -1).bfloat16().cuda(), idx, off


# Query heads (key-value heads as many), sequences, length, first position of the window, candidates of a sequence: tiles of 64
# rows for update and exact rows, and of 128 (more than 80 rows a sequence); sequences without candidates, with a tile that is
# full and with several.
@pytest.mark.parametrize("heads,B,L,row_lo,counts", [(32, 4, 300, 230, [5, 64, 0, 1]), (32, 4, 300, 236, [64, 64, 40, 64]),
                                                     (32, 4, 400, 0, [90, 128, 100, 129]), (32, 5, 300, 100, [0, 200, 150, 81, 60]),
                                                     (16, 8, 257, 0, [100, 81, 1, 128, 200, 90, 90, 90])])
def test_exact_rows_beside_the_update(heads, B, L, row_lo, counts):
    print("update and exact rows", heads, B, L, row_lo, counts, flush=True)
    s = W.LayerShape(hidden=512, n_heads=heads, n_kv_heads=heads, head_dim=128, ffn=512, dtype="bf16")
    x0, x1, idx, off = _inputs(s, B, L, row_lo, counts, 91)
    w = rand_weights(s, 92, bias=True)
    res = []
    for keep_lse in (False, True):
        lay = Layer.from_shape(s, B, L, keep_lse=keep_lse)
        lay.set_weights(w)
        lay.full_step(x0)
        if res:
            for name, t in zip(CACHES, start):  # (the dense step of such a layer has another merge too)
                getattr(lay, name).copy_(t)
        start = [getattr(lay, name).clone() for name in CACHES]
        out = lay.layer_step_approx(x1, lay.make_list(idx, off), -2.0, row_lo=row_lo)  # (nothing falls below tau: contexts alone)
        assert int(out.offsets[-1]) == 0
        res.append([getattr(lay, name).clone() for name in CACHES])
        lay.close()
    (k0, v0, c0, o0), (k1, v1, c1, o1) = res
    assert torch.equal(k0, k1) and torch.equal(v0, v1) and torch.equal(o0, o1)
    cand = torch.zeros(B * L, dtype=torch.bool, device="cuda")
    cand[torch.from_numpy(idx).long().cuda()] = True
    c0, c1, cs = c0.view(B * L, -1), c1.view(B * L, -1), start[2].view(B * L, -1)
    assert torch.equal(c0[~cand], c1[~cand]) and not torch.equal(c0[~cand], cs[~cand])
    # exact rows: the sums of the same tiles, divided by the row sum before they are stored or in the merge (fp32 rounding, which
    # moves one value in some thousands to the next of its 8 bits)
    a, b = c0[cand].float(), c1[cand].float()
    assert ((a - b).abs() <= 2.0 ** -7 * a.abs().clamp_min(1e-30)).all()
    assert (a != b).float().mean().item() < 1e-2 and not torch.equal(c0[cand], cs[cand])


@pytest.mark.parametrize("shape,approx", [("mha", 1), ("mha", 2), ("dh64", 1), ("grouped", 1)])
@pytest.mark.parametrize("B,L,row_lo,counts", [(1, 700, 400, [70]), (3, 500, 300, [20, 200, 77]), (2, 300, 44, [129, 256])])
def test_candidates_share_the_rows_normalised_for_q(shape, approx, B, L, row_lo, counts):
    print("shared rows", shape, approx, B, L, counts, flush=True)
    s = {"mha": W.LayerShape(hidden=512, n_heads=4, n_kv_heads=4, head_dim=128, ffn=512, dtype="bf16"),
         "dh64": W.LayerShape(hidden=256, n_heads=4, n_kv_heads=2, head_dim=64, ffn=384, dtype="bf16"),
         "grouped": W.LayerShape(hidden=1024, n_heads=14, n_kv_heads=2, head_dim=128, ffn=512, dtype="bf16")}[shape]
    x0, x1, idx, off = _inputs(s, B, L, row_lo, counts, 93)
    w = rand_weights(s, 94, bias=True)
    res = []
    for loop in (False, True):
        st = Stack(s, 1, B, L, keep_lse=approx == 2)
        lay = st.layers[0]
        lay.set_weights(w)
        st.full_step(x0)
        if loop:
            cand = Bd.IndexList.empty(B * L, B)
            kind, out = st.denoise_step(Bd.Schedule(1, 4, row_lo, approx, 0.97), 5, x1, lay.make_list(idx, off), None, cand)
            assert kind == Bd.STEP_RESPONSE and cand.offsets.tolist() == off.tolist()
        else:
            # (the merged list has room for all tokens; so has this one, for the same plans)
            out = lay.layer_step_approx(x1, lay.make_list(idx, off, cap=B * L), 0.97, row_lo=row_lo, cached_norm=approx == 2)
        n = int(out.offsets[-1])
        res.append([getattr(lay, name).clone() for name in CACHES] + [out.offsets.clone(), out.idx[:n].clone()])
        assert n > 0
        st.close()
    for name, a, b in zip(CACHES + ("offsets", "idx"), *res):
        assert torch.equal(a, b), name
