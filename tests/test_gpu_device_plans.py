"""Plans made on the device (a list's count is there alone) against those of the host planner, which the CPU tests look at:
another implementation, a candidate per lane, prices cut to 17 bits, four waves that exchange their least through LDS."""
import ctypes as C
import os

import numpy as np
import pytest

from paper_2603_08026_amd import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    torch.cuda.init()
    if not os.path.exists(build.PROBE):
        build.build_probe()
    return C.CDLL(build.PROBE)


@pytest.mark.parametrize("kind", ["raw", "gate_up", "down"])
@pytest.mark.parametrize("n,k", [(12288, 4096), (4096, 4096), (4608, 3584), (1536, 512), (3072, 1024), (2048, 2048), (14336, 4096)])
def test_plans_of_the_device_are_those_of_the_host(lib, kind, n, k):
    print("device plans", kind, n, k, flush=True)
    if kind == "down":
        n, k = k, n
    rng = np.random.default_rng(7)
    rows = np.concatenate([np.arange(0, 1200, 3), np.round(np.exp(rng.uniform(np.log(120), np.log(40000), 1600)))]).astype(np.int32)
    out = (C.c_int * 6)()
    rc = lib.compare_plans({"raw": 0, "gate_up": 1, "down": 2}[kind], n, k, C.c_long(1 << 28), rows.size,
                           rows.ctypes.data_as(C.POINTER(C.c_int)), out)
    assert rc == 0
    differ, wrong, cols128, cols256, cols192, at = out
    assert wrong == 0, at
    assert differ < rows.size // 50  # (equal prices to 17 bits)
    assert cols128 + cols256 + cols192 == rows.size
