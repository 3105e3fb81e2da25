"""List unions on both sides of the token count up to which one launch does it all: a single token, chunk
edges (256 tokens), the last count of the one-launch form and the first beyond it; empty, full and disjoint
lists.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from tests.helpers import rand_rows, small_shape
from oracle import dyllm_oracle as O
from paper_2603_08026_amd import binding
from paper_2603_08026_amd.layer import Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L", [(1, 1), (1, 255), (2, 128), (1, 257), (3, 300), (2, 4096), (1, 8193)])
def test_union_in_one_launch_and_in_four(B, L):
    print("merge lists", B, L, flush=True)
    lay = Layer.from_shape(small_shape("bf16"), B, L)
    out = binding.IndexList.empty(B * L, B)
    for na, nb, lo in ((0, 0, 0), (1, 0, 0), (L // 2, L // 3, 0), (L, L // 5, L // 4), (L, L, 0)):
        a, aoff = rand_rows(71, B, L, [na] * B)
        b, boff = rand_rows(72, B, L, [nb] * B)
        lay.ctx.merge_lists(lay.make_list(a, aoff, cap=B * L), lay.make_list(b, boff), B, L, lo, out)
        torch.cuda.synchronize()
        want = O.merge_lists(a, b, L, lo)
        idx, off = lay.read_list(out)
        assert np.array_equal(idx, want), (na, nb, lo)
        assert np.array_equal(off, np.searchsorted(want, np.arange(B + 1) * L)), (na, nb, lo)
    lay.close()
