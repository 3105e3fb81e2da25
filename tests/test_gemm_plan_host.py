"""The bf16 GEMMs' launch rules (gemm_plan.h), compiled for the host: no GPU needed."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2603_08026_amd import build

SOURCE = r"""
#include "%s/gemm_plan.h"
using namespace dy::mm;
extern "C" int groups_ok(int end0, int end1) { return ring_groups_ok(end0, end1); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE % build.CSRC)
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared",
                        "-fPIC", src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return C.CDLL(so)


@pytest.mark.parametrize("end", [8, 16, 24, 40, 4096 + 8, 4096 + 16])
def test_matrix_ends_inside_a_group_of_permuted_rows_are_not_for_the_ring_loop(lib, end):
    assert not lib.groups_ok(end, 8192)
    assert not lib.groups_ok(4096, end)


@pytest.mark.parametrize("dq,dkv", [(4096, 4096), (3584, 512), (256, 64), (128, 128)])
def test_ends_of_the_stacked_projections_are(lib, dq, dkv):
    assert lib.groups_ok(dq, dq + dkv)
    assert lib.groups_ok(dkv, 2 * dkv)
