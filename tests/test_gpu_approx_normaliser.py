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
