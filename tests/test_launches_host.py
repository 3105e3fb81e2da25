"""The launches of whole calls, recorded without a GPU (launch_probe.hip): every GEMM and row kernel that reads a plan from device memory finds there
the plan that was made for it."""
import os
import subprocess

import pytest

from paper_2603_08026_amd import binding, build
from tests.test_gpu_attention_tiles import SWEEP, sweep_lists
from tests.test_gpu_listed_steps import COMMITTED

SHAPES = {  # hidden, query heads, KV heads, head_dim, FFN width
    "8b": (4096, 32, 32, 128, 12288),
    "7b": (3584, 28, 4, 128, 18944),
    "split down": (512, 4, 2, 128, 4096),
    "no sums": (512, 8, 8, 64, 640),
}


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    exe = str(tmp_path_factory.mktemp("launch") / "probe")
    d, so = os.path.split(binding.LIB_PATH)
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-O1", "-rdynamic", os.path.join(build.TESTS, "launch_probe.hip"), "-o", exe, "-L" + d, "-l:" + so,
                        "-Wl,-rpath," + d], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def launches(probe, case, cap, shape, B=3, L=900, lo=0, cached=0):
    args = [probe, case] + [str(v) for v in (cap, *SHAPES.get(shape, shape), B, L, lo, cached)]
    r = subprocess.run(args, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    out = []
    for line in r.stdout.splitlines():
        name, *words = line.split(" ")
        out.append((name, [tuple(w.split("=")) for w in words]))
    return out


def check(events):
    """A plan is made (by a row kernel, or by a GEMM for itself), read by the GEMM it was made for, and by the row kernel behind that GEMM;
    nothing else is put in its place in between.  Returns how many GEMMs read a plan made ahead."""
    held, reads, last = {}, 0, None  # words -> (launch that made the plan, GEMM that has run by it)
    for i, (name, words) in enumerate(events):
        for what, at in words:
            assert at not in ("0", "(nil)"), (i, name, what)  # a plan from nowhere
            if what == "reads":
                assert at in held and held[at][1] is None, (i, name, "reads a plan that another GEMM has used or nobody has made")
                held[at] = (held[at][0], i)
                last = at
                reads += 1
            elif what == "splits":
                assert at == last and held[at][1] is not None, (i, name, "reads the splits of another GEMM")
            else:
                assert at not in held or held[at][1] is not None, (i, name, "a plan was made and nobody has read it")
                gemm = "k_gemm_planned" in name
                held[at] = (i, i if gemm else None)
                if gemm:
                    last = at
    assert all(gemm is not None for _, gemm in held.values()), "a plan that nobody reads"
    return reads


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("cap", [100, 200, 300, 1000, 2700])
@pytest.mark.parametrize("case,lo,cached", [("step", 0, 0), ("ffn", 0, 0), ("approx", 0, 0), ("approx", 700, 0), ("approx", 0, 1),
                                            ("approx", 700, 1)])
def test_plans_reach_their_gemms(probe, shape, cap, case, lo, cached):
    ahead = check(launches(probe, case, cap, shape, lo=lo, cached=cached))
    assert ahead == (0 if cap <= 256 else 2 if case == "ffn" else 3)


# The norm kernel leaves the plan of the candidates' k and v ahead of the GEMM for q of all tokens: that GEMM makes a plan of its own where
# the device counts its rows.
@pytest.mark.parametrize("cached", [0, 1])
@pytest.mark.parametrize("shape", ["8b", "split down"])
def test_candidates_plan_outlasts_the_query_projection(probe, shape, cached):
    assert check(launches(probe, "counted window", 1000, shape, lo=500, cached=cached)) == 3

# A GEMM that cannot plan for itself and gets no plan takes tiles that need none.
@pytest.mark.parametrize("case", ["down alone", "up alone"])
@pytest.mark.parametrize("cap", [300, 2700])
def test_gemm_without_a_plan(probe, case, cap):
    events = launches(probe, case, cap, "8b")
    assert events and not any("k_gemm_planned" in name for name, _ in events), events


def attention_plan(probe, heads, kv, B, L, cap):
    """Rows in a query tile, key splits, key tiles of the first split, whether a last tile is not full."""
    (_, words), = launches(probe, "attention", cap, (128, heads, kv, 128, 128), B=B, L=L)
    p = {k: int(v) for k, v in words}
    tile = 32 if p["bq"] == 128 else 64
    keys = min(L, p["chunk"])
    return p["bq"], p["splits"], -(-keys // tile), keys % tile > 0


def test_attention_sweep_runs_what_it_names(probe):
    """Key tiles of the cases whose rows are finished in place, for both kernels; a case of several heads to a group in each, with a steady state
    that is unrolled and a last tile that is not full; and cases that are cut over keys."""
    seen, grouped, split = {64: {}, 128: {}}, set(), 0
    for heads, kv, times, L in SWEEP:
        idx, off, caps = sweep_lists(heads, kv, times, L)
        for cap in caps:
            bq, splits, tiles, partial = attention_plan(probe, heads, kv, off.size - 1, L, cap)
            if splits > 1:
                split += 1
                continue
            seen[bq].setdefault(tiles, set()).add(partial)
            if heads > kv and tiles > 8 and partial:
                grouped.add(bq)
    for bq in (64, 128):
        assert set(range(1, 11)) <= set(seen[bq]), (bq, sorted(seen[bq]))
        assert any(n >= 12 for n in seen[bq])
        assert sum(len(p) == 2 for p in seen[bq].values()) >= 3, seen[bq]
    assert grouped == {64, 128} and split >= 10


@pytest.mark.parametrize("name", COMMITTED)
def test_committed_rows_run_what_they_name(probe, name):
    s, L, counts = COMMITTED[name]
    B = len(counts)
    for cap, bq in ((sum(counts), 64), (B * L, 128)):
        assert attention_plan(probe, s.n_heads, s.n_kv_heads, B, L, cap)[:2] == (bq, 1)
