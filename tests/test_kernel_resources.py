"""Row kernels of 1024 threads: two workgroups to a CU, as their grids count on, by the compiler's own resource figures.  No GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2603_08026_amd import build


@pytest.fixture(scope="module")
def figures():
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "rowops.hip"), "-o", os.devnull,
                        "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark: (?:.*remark: )?\s*(Function Name|TotalSGPRs|VGPRs|Occupancy \[waves/SIMD\]|SGPRs Spill|VGPRs Spill): (\S+)", line)
        if not m:
            continue
        if m.group(1) == "Function Name":
            name = m.group(2)
            out[name] = {}
        else:
            out[name][m.group(1).split(" [")[0]] = int(m.group(2))
    return out


# A workgroup is 16 waves, four to a SIMD: two of them need eight.  (bf16; k_qkv_finalize without candidates)
@pytest.mark.parametrize("kernel", ["k_qkv_finalizeItLNS_8DvLayoutE0E", "k_oproj_finalizeILb0E", "k_oproj_finalizeILb1E", "k_down_finalize"])
def test_two_workgroups_to_a_cu(figures, kernel):
    found = [f for n, f in figures.items() if kernel in n]
    assert len(found) == 1, sorted(figures)
    f = found[0]
    assert f["Occupancy"] == 8 and f["SGPRs Spill"] == 0 and f["VGPRs Spill"] == 0, f


# the forms with candidates: no vector register goes to memory
@pytest.mark.parametrize("layout", [1, 2, 3])
def test_candidates(figures, layout):
    found = [f for n, f in figures.items() if "k_qkv_finalizeItLNS_8DvLayoutE%dE" % layout in n]
    assert len(found) == 1 and found[0]["Occupancy"] >= 7 and found[0]["VGPRs Spill"] == 0, found
