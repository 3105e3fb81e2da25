"""Plans that a row kernel makes for the GEMMs behind it: calls with other counts before them leave other plans in the same words,
so every call on a context that has seen all counts is compared bit by bit with the same call on a fresh one, whose words are zero
(another plan has other K splits or leaves rows out).  Counts in the weight-streaming tiles, at their edge, in one row tile and in several."""
import pytest
import torch

from paper_2603_08026_amd import binding as Bd
from paper_2603_08026_amd.layer import Layer
from synth import workload as W
from tests.helpers import rand_rows, rand_weights

pytestmark = pytest.mark.gpu

SHAPES = {
    "split down": W.LayerShape(hidden=512, n_heads=4, n_kv_heads=2, head_dim=128, ffn=4096, dtype="bf16"),
    "no sums": W.LayerShape(hidden=512, n_heads=8, n_kv_heads=8, head_dim=64, ffn=640, dtype="bf16"),
    "wide": W.LayerShape(hidden=2048, n_heads=16, n_kv_heads=4, head_dim=128, ffn=2816, dtype="bf16"),
}
B, L = 3, 900
COUNTS = [40, 1500, 128, 129, 600, 2700, 330, 0, 260]


def _caches(lay):
    return [lay.k, lay.v, lay.c, lay.out]


# approx: the first position of the approximate step (0: whole sequences, else a response window; listed tokens ahead of it get k and v alone),
# or no such step
@pytest.mark.parametrize("approx", [None, 0, 500])
@pytest.mark.parametrize("name", SHAPES)
def test_other_counts_before(name, approx):
    print("plans ahead", name, approx, flush=True)
    s, T = SHAPES[name], B * L
    w = rand_weights(s, 61, bias=True)
    gen = torch.Generator().manual_seed(62)
    xs = [torch.randn(B, L, s.hidden, generator=gen).to(torch.bfloat16).cuda() for _ in range(2)]

    def layer():
        lay = Layer.from_shape(s, B, L)
        lay.set_weights(w)
        return lay

    used = layer()
    used.full_step(xs[0])
    start = [t.clone() for t in _caches(used)]
    for count in COUNTS:
        idx, off = rand_rows(63, B, L, [count // B + (1 if b < count % B else 0) for b in range(B)])
        got = []
        for lay in (used, layer()):
            for t, t0 in zip(_caches(lay), start):
                t.copy_(t0)
            rows = lay.make_list(idx, off, cap=T)
            if approx is None:
                out = lay.layer_step(xs[1], rows, 0.9, Bd.IndexList.empty(T, B))
            else:
                out = lay.layer_step_approx(xs[1], rows, 0.9, Bd.IndexList.empty(T, B), row_lo=approx)
            got.append([t.clone() for t in _caches(lay)] + [out.offsets.clone()])
            assert lay.ctx.poll_status() == 0
            if lay is not used:
                lay.close()
        for a, b in zip(*got):
            assert torch.equal(a, b), count
    used.close()
