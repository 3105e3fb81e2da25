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


# Rows that the attention kernel commits: a wait for loads also waits for the stores before it, so no wait stands between the stores of the rows of a
# wave (with one behind each, launches of one item a CU took 1 to 1.5 us more).  The listing of every kernel has the stores of partial results, then
# those of the rows: a wait between the two groups at most (in each of the forms that a kernel holds).
def test_no_wait_between_the_rows_that_are_committed(tmp_path):
    asm = str(tmp_path / "attention.s")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "attention_bf16.hip"), "-o", asm],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels, name = {}, None
    for line in open(asm):
        m = re.match(r"(_ZN2dy\w*k_attn_bf16_(?:dma|both)\w*):", line)
        if m:
            name = m.group(1)
            kernels[name] = ""
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and re.search(r"global_store_dwordx4", line):
            kernels[name] += "s"
        elif name and re.search(r"s_waitcnt.*vmcnt", line):
            kernels[name] += "w"
    assert len(kernels) == 8
    for name, order in kernels.items():
        forms = 2 if "both" in name or "OnceE2" in name else 1
        assert len(re.findall(r"s(?=w+s)", order)) <= 2 * forms, (name, order)
        assert order.count("s") >= 24 * forms, (name, order)  # (16 and 8)
