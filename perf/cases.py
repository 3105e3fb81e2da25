"""The work that is timed: what a user of this library has it do, through its public entry points.

A pass of every sparse case works on caches that an earlier step left, as in the generation loop: the
inputs alternate between two versions of the hidden states, so that the same tokens are salient again in
every pass.  Of the candidates a share `kept` has really moved (redrawn, as in the benchmark) and falls
below tau; the others are candidates that have settled, which the cosine test drops.  Weights are
random-init, hidden states N(0, 1), as everywhere in this repository.  Such layers lack the temporal
stability of a trained model: with a quarter of the keys redrawn a settled token's context still keeps a
cosine of about 0.75, a redrawn token's falls to 0.3 or less, so tau stands between the two.
"""
import math

import torch

from paper_2603_08026_amd import binding
from paper_2603_08026_amd.layer import Layer, Stack, torch_dtype
from synth.workload import DREAM, LLADA, TINY, LayerShape

SHAPES = {
    "llada": LLADA,   # 8B layer, 32 heads
    "dream": DREAM,   # 7B layer, 28 query heads over 4 KV heads
    "tiny": TINY,     # fp32, head_dim 64
    "small": LayerShape(hidden=512, n_heads=8, n_kv_heads=2, head_dim=64, ffn=1536, dtype="bf16"),  # bf16, head_dim 64
}
TAU = 0.5
RESP = 256     # response positions of a sequence (the last ones)


def listed():
    return [
        # one tiny fp32 layer: what is left of a step when there is next to nothing to compute
        dict(name="tiny-f32-step", kind="step", shape="tiny", batch=1, seq=128, frac=0.10, kept=0.8),
        # interactive use: one request, a tenth of its 1024 tokens; weights dominate
        dict(name="b1-step-10pct", kind="step", shape="llada", batch=1, seq=1024, frac=0.10, kept=0.8),
        # serving batch at the salient share of trained models (1.3 - 8.4 % per layer)
        dict(name="b16-step-2pct", kind="step", shape="llada", batch=16, seq=1280, frac=0.02, kept=0.8),
        # the benchmark's workload, and the upper end of its sweep
        dict(name="b16-step-10pct", kind="step", shape="llada", batch=16, seq=1280, frac=0.10, kept=1.0),
        dict(name="b16-step-25pct", kind="step", shape="llada", batch=16, seq=1280, frac=0.25, kept=1.0),
        # grouped heads (28 over 4), odd request count and length
        dict(name="gqa-b13-step-7pct", kind="step", shape="dream", batch=13, seq=1277, frac=0.07, kept=0.9),
        # dense warm-up steps: one request, and the serving batch
        dict(name="b1-dense", kind="dense", shape="llada", batch=1, seq=1024),
        dict(name="b16-dense", kind="dense", shape="llada", batch=16, seq=1280),
        # several layers in one call, long sequences
        dict(name="stack3-b16-10pct", kind="stack", shape="llada", batch=16, seq=2048, frac=0.10, kept=0.9, layers=3),
        # the generation loop: four steps (one whole-sequence, three response-only) with the carried set;
        # how many tokens are salient is known to the device alone
        dict(name="loop-exact-b8", kind="loop", shape="llada", batch=8, seq=1024, frac=0.04, kept=1.0, layers=2, approx=0),
        dict(name="loop-approx-b8", kind="loop", shape="llada", batch=8, seq=1024, frac=0.04, kept=1.0, layers=2, approx=1),
        # the salient test alone, over all tokens of a batch
        dict(name="saliency-all-tokens", kind="saliency", shape="llada", batch=16, seq=2048, frac=0.10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "dense", "stack", "loop", "saliency"])
    shape = rng.choice(["llada", "llada", "llada", "dream", "dream", "small", "tiny"]) if kind == "step" else rng.choice(["llada", "dream"])
    big = shape in ("llada", "dream")
    batch = _log_int(rng, 1, 16 if big else 4)
    seq = _log_int(rng, 384, 2048 if batch <= 10 else 1280) if big else _log_int(rng, 96, 768)
    c = dict(kind=kind, shape=shape, batch=batch, seq=seq)
    if kind == "dense":
        return c
    c["frac"] = round(math.exp(rng.uniform(math.log(0.01), math.log(0.25 if kind == "step" else 0.10))), 4)
    if kind == "saliency":
        return c
    c["kept"] = round(rng.uniform(0.7, 1.0), 2) if c["frac"] <= 0.12 else 1.0  # (a settled token stays far from tau)
    if kind == "stack":
        c["layers"] = rng.randint(2, 3)
    if kind == "loop":
        c["layers"], c["approx"] = 2, rng.choice([0, 1, 2])
        c["batch"], c["frac"] = min(batch, 8), min(c["frac"], 0.05)
    if kind == "step" and shape == "dream":
        c["bias"] = rng.random() < 0.5
    return c


# ---- inputs -------------------------------------------------------------------------------------------

def _per_seq(case):
    """Candidates of every sequence (ragged: 0.5 .. 1.5 times the share) and how many of them have moved."""
    B, L = case["batch"], case["seq"]
    span = min(RESP, L // 2) if case["kind"] == "loop" else L  # the loop's carried set lies in the response
    out = []
    for b in range(B):
        r = 0.5 + ((b * 0.6180339887) % 1.0) if B > 1 else 1.0
        n = min(span, max(1, round(case["frac"] * L * r)))
        out.append((n, max(1, round(n * case.get("kept", 1.0)))))
    return out, span


def _weights(s, gen, bias):
    td = torch_dtype(s.dtype)
    std = 0.02 * math.sqrt(4096.0 / s.hidden)
    d, dq, dkv, f = s.hidden, s.dq, s.dkv, s.ffn
    def mat(n, k):
        return torch.empty(n, k, dtype=td, device="cuda").normal_(0.0, std, generator=gen)
    w = dict(wq=mat(dq, d), wk=mat(dkv, d), wv=mat(dkv, d), wo=mat(d, dq), w_gate=mat(f, d), w_up=mat(f, d), w_down=mat(d, f))
    for n in ("g_attn", "g_ffn"):
        w[n] = (1.0 + 0.1 * torch.randn(d, device="cuda", generator=gen)).to(td)
    if bias:
        for n, k in (("bq", dq), ("bk", dkv), ("bv", dkv)):
            w[n] = (0.1 * torch.randn(k, device="cuda", generator=gen)).to(td)
    return w


def _hidden(s, B, L, gen):
    return torch.randn(B * L, s.hidden, device="cuda", generator=gen).to(torch_dtype(s.dtype))


def _candidates(case, gen_cpu):
    """(all candidates, the moved ones among them, per-sequence offsets of the former), flat token ids."""
    B, L = case["batch"], case["seq"]
    counts, span = _per_seq(case)
    cand, moved, off = [], [], [0]
    for b, (n, m) in enumerate(counts):
        p = torch.randperm(span, generator=gen_cpu)[:n] + (L - span)
        cand.append(torch.sort(p)[0] + b * L)
        moved.append(torch.sort(p[:m])[0] + b * L)
        off.append(off[-1] + n)
    return torch.cat(cand), torch.cat(moved), off


def _index_list(ids, off, cap=None):
    buf = torch.zeros(int(ids.numel()) if cap is None else cap, dtype=torch.int32)
    buf[:ids.numel()] = ids.to(torch.int32)
    return binding.IndexList(buf.cuda(), torch.tensor(off, dtype=torch.int32).cuda())


def _inputs(case, seed):
    """Everything that is drawn for a case: plain tensors on the GPU (the lists on the CPU)."""
    s, B, L, kind = SHAPES[case["shape"]], case["batch"], case["seq"], case["kind"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    gen_cpu = torch.Generator().manual_seed(seed)
    if kind == "saliency":
        ids, _, _ = _candidates(case, gen_cpu)
        ids = ids.cuda()
        old = torch.randn(B * L, s.dq, device="cuda", generator=gen)
        new = old + 0.02 * torch.randn(B * L, s.dq, device="cuda", generator=gen)
        new[ids] = torch.randn(ids.numel(), s.dq, device="cuda", generator=gen)
        return dict(old=old.to(torch_dtype(s.dtype)), new=new.to(torch_dtype(s.dtype)))
    d = dict(weights=[_weights(s, gen, case.get("bias", False)) for _ in range(case.get("layers", 1))])
    x0 = _hidden(s, B, L, gen)
    d["x"] = [x0]
    if kind == "dense":
        return d
    ids, moved, off = _candidates(case, gen_cpu)
    x1 = x0.clone()
    at = moved.cuda()
    x1[at] = torch.randn(at.numel(), s.hidden, device="cuda", generator=gen).to(x0.dtype)
    d["x"].append(x1)
    d.update(ids=ids, moved=moved, off=off)
    if kind == "loop":
        # one token per sequence has just been decoded (a moved one); the rest is carried
        starts = [0]
        for _, m in _per_seq(case)[0]:
            starts.append(starts[-1] + m)
        d["decoded"] = moved[torch.tensor(starts[:-1])]
    return d


def prepare(case, seed):
    torch.cuda.set_device(0)
    s, B, L, kind = SHAPES[case["shape"]], case["batch"], case["seq"], case["kind"]
    d = _inputs(case, seed)
    st = dict(kind=kind, B=B, L=L, turn=0)
    if kind == "saliency":
        lay = Layer.from_shape(s, 1, 1)  # (a context for the calls; max_batch and max_seq below)
        cfg = binding.LayerCfg(s.hidden, s.n_heads, s.n_kv_heads, s.head_dim, s.ffn, B, L, B * L, lay.cfg.dtype, s.rms_eps, s.rope_theta)
        lay.close()
        st.update(ctx=binding.Context(cfg), old=d["old"], new=d["new"],
                  cos=torch.zeros(B * L, device="cuda"), flag=torch.zeros(B * L, dtype=torch.uint8, device="cuda"),
                  out=binding.IndexList.empty(B * L, B))
        return st
    n_layers = case.get("layers", 1)
    if n_layers == 1 and kind in ("step", "dense"):
        one = Layer.from_shape(s, B, L)
        layers, st["layer"] = [one], one
    else:
        stack = Stack(s, n_layers, B, L, keep_lse=case.get("approx") == 2)
        layers, st["stack"] = stack.layers, stack
    for lay, w in zip(layers, d["weights"]):
        lay.set_device_weights(w)
    st["x"] = [x.view(B, L, -1) for x in d["x"]]
    if kind == "dense":
        return st
    # the dense step before: it fills the caches
    if "layer" in st:
        st["layer"].full_step(st["x"][0])
        st["idx"] = _index_list(d["ids"], d["off"])
        st["layer"].idx_out = binding.IndexList.empty(st["idx"].cap, B)
    else:
        st["stack"].full_step(st["x"][0])
        if kind == "stack":
            st["idx"] = _index_list(d["ids"], d["off"])
        else:
            st["decoded"] = _index_list(d["decoded"], list(range(B + 1)))
            st["carry"] = _index_list(d["ids"], d["off"], cap=B * L)
            st["cand"] = binding.IndexList.empty(B * L, B)
            st["sched"] = binding.Schedule(1, 4, L - min(RESP, L // 2), case["approx"], TAU)
    return st


def _caches(layers):
    return [dict(k=l.k, v=l.v, c=l.c, out=l.out) for l in layers]


def run(st):
    kind = st["kind"]
    if kind == "saliency":
        st["ctx"].saliency(st["new"], st["old"], None, st["B"], st["L"], TAU, st["cos"], st["flag"])
        st["ctx"].compact(st["flag"], None, st["B"], st["L"], st["out"])
        return dict(cos=st["cos"], flag=st["flag"], idx=st["out"].idx, offsets=st["out"].offsets)
    if kind == "dense":
        st["layer"].full_step(st["x"][0])
        return _caches([st["layer"]])
    if kind == "loop":
        stack, carry = st["stack"], st["carry"]
        for t in range(4, 8):  # t = 4: whole sequence, 5 .. 7: response only
            st["turn"] ^= 1
            _, carry = stack.denoise_step(st["sched"], t, st["x"][st["turn"]], st["decoded"], carry, st["cand"])
        return dict(caches=_caches(stack.layers), carry=carry.offsets, cand=st["cand"].offsets)
    st["turn"] ^= 1
    x = st["x"][st["turn"]]
    if kind == "stack":
        outs = st["stack"].stack_step(x, st["idx"], TAU)
        n = len(st["stack"].layers) * st["idx"].cap
        return dict(caches=_caches(st["stack"].layers), cos=st["stack"].cos.view(-1)[:n], offsets=[o.offsets for o in outs])
    out = st["layer"].layer_step(x, st["idx"], TAU)
    return dict(caches=_caches([st["layer"]]), cos=st["layer"].cos[:st["idx"].cap], idx=out.idx, offsets=out.offsets)


# ---- the same pass in 64 bits: plain torch, nothing rounded in between ------------------------------------

def _norm64(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _heads64(s, x, w, b, n_heads, rows, L, rotate):
    y = x @ w.t()
    if b is not None:
        y = y + b
    y = y.view(-1, n_heads, s.head_dim)
    if rotate:
        half = s.head_dim // 2
        freq = s.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / s.head_dim)
        a = ((rows % L).double()[:, None] * freq)[:, None, :]
        lo, hi = y[..., :half], y[..., half:]
        y = torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)
    return y


def _attend64(s, q, rows, k, v, L):
    """Attention rows of the queries at tokens `rows` over k, v [B*L, Hkv, dh] of their sequences."""
    out = torch.empty(rows.numel(), s.n_heads, s.head_dim, dtype=torch.float64, device="cuda")
    g = s.n_heads // s.n_kv_heads
    for b in torch.unique(rows // L).tolist():
        at = (rows // L == b).nonzero().view(-1)
        kb, vb = k[b * L:(b + 1) * L], v[b * L:(b + 1) * L]
        for h in range(s.n_kv_heads):
            p = torch.softmax(q[at, h * g:(h + 1) * g].reshape(-1, s.head_dim) @ kb[:, h].t() / math.sqrt(s.head_dim), -1)
            out[at, h * g:(h + 1) * g] = (p @ vb[:, h]).view(-1, g, s.head_dim)
    return out.view(rows.numel(), -1)


def _layer64(s, w, c, x, rows, L, window=None):
    """One layer over the tokens `rows` (updates the caches c); returns their cosines and the tokens below tau.
    window: also update the contexts of these tokens through the changed values of `rows`."""
    n = _norm64(x[rows], w["g_attn"], s.rms_eps)
    q = _heads64(s, n, w["wq"], w.get("bq"), s.n_heads, rows, L, True)
    v = _heads64(s, n, w["wv"], w.get("bv"), s.n_kv_heads, rows, L, False)
    dv = torch.zeros_like(c["v"])
    dv[rows] = v - c["v"][rows]
    c["k"][rows] = _heads64(s, n, w["wk"], w.get("bk"), s.n_kv_heads, rows, L, True)
    c["v"][rows] = v
    exact_rows = _attend64(s, q, rows, c["k"], c["v"], L)
    toks, new = rows, exact_rows
    if window is not None:
        toks = window
        qa = _heads64(s, _norm64(x[toks], w["g_attn"], s.rms_eps), w["wq"], w.get("bq"), s.n_heads, toks, L, True)
        full = c["c"].clone()
        full[toks] += _attend64(s, qa, toks, c["k"], dv, L)
        full[rows] = exact_rows
        new = full[toks]
    old = c["c"][toks]
    cos = (new * old).sum(-1) / (new.norm(dim=-1).clamp_min(1e-8) * old.norm(dim=-1).clamp_min(1e-8))
    c["c"][toks] = new
    return cos, toks[cos < TAU]


def _ffn64(s, w, c, x, rows):
    h = x[rows] + c["c"][rows] @ w["wo"].t()
    f = _norm64(h, w["g_ffn"], s.rms_eps)
    c["out"][rows] = h + (torch.nn.functional.silu(f @ w["w_gate"].t()) * (f @ w["w_up"].t())) @ w["w_down"].t()


def exact(case, seed):
    if case.get("approx") == 2:
        return None  # (the carried normalisers make this form's result depend on the steps before)
    torch.cuda.set_device(0)
    s, B, L, kind = SHAPES[case["shape"]], case["batch"], case["seq"], case["kind"]
    d = _inputs(case, seed)
    if kind == "saliency":
        a, b = d["new"].double(), d["old"].double()
        return dict(cos=(a * b).sum(-1) / (a.norm(dim=-1) * b.norm(dim=-1)), flag=None, idx=None, offsets=None)
    T, n_layers = B * L, case.get("layers", 1)
    W = [{k: v.double() for k, v in w.items()} for w in d["weights"]]
    X = [x.double() for x in d["x"]]
    def zeros(*sh):
        return torch.zeros(T, *sh, dtype=torch.float64, device="cuda")
    C = [dict(k=zeros(s.n_kv_heads, s.head_dim), v=zeros(s.n_kv_heads, s.head_dim), c=zeros(s.dq), out=zeros(s.hidden)) for _ in W]
    every = torch.arange(T, device="cuda")
    x = X[0]
    for w, c in zip(W, C):
        _layer64(s, w, c, x, every, L)
        _ffn64(s, w, c, x, every)
        x = c["out"]
    cos = None
    def step(x, rows, window=None):
        for w, c in zip(W, C):
            cs, rows = _layer64(s, w, c, x, rows, L, window)
            _ffn64(s, w, c, x, rows)
            x = c["out"]
        return cs, rows
    if kind == "loop":
        carry, dec, lo = d["ids"].cuda(), d["decoded"].cuda(), L - min(RESP, L // 2)
        for t in range(4, 8):
            win = every if t % 4 == 0 else every[every % L >= lo]
            rows = torch.unique(torch.cat([carry, dec]))
            rows = rows if t % 4 == 0 else rows[rows % L >= lo]
            _, carry = step(X[(t + 1) % 2], rows, win if case["approx"] else None)
    elif kind != "dense":
        cos, _ = step(X[1], d["ids"].cuda())
    caches = [dict(k=c["k"].view(B, L, s.n_kv_heads, -1), v=c["v"].view(B, L, s.n_kv_heads, -1), c=c["c"].view(B, L, -1),
                   out=c["out"].view(B, L, -1)) for c in C]
    if kind == "dense":
        return caches
    if kind == "loop":
        return dict(caches=caches, carry=None, cand=None)
    if kind == "stack":
        return dict(caches=caches, cos=None, offsets=[None] * n_layers)
    return dict(caches=caches, cos=cos, idx=None, offsets=None)


# ---- what a pass cannot do without ----------------------------------------------------------------------

def work(case):
    s, B, L = SHAPES[case["shape"]], case["batch"], case["seq"]
    e = 4 if s.dtype == "f32" else 2
    T, d, dq, dkv, f = B * L, s.hidden, s.dq, s.dkv, s.ffn
    if case["kind"] == "saliency":
        return {"bytes": 2.0 * T * dq * e + T * 5, "flops": 6.0 * T * dq}
    w_bytes = float((dq + 2 * dkv) * d + d * dq + 3 * f * d) * e
    def layer(m, m_out, dense):
        flops = 2.0 * m * d * (dq + 2 * dkv) + 4.0 * m * L * dq + m_out * (2.0 * dq * d + 6.0 * d * f)
        rows = m * (d + 2 * dkv + dq) + m_out * d + (0 if dense else 2 * T * dkv + m * dq)
        return w_bytes + float(rows) * e, flops
    if case["kind"] == "dense":
        b, fl = layer(T, T, True)
        return {"bytes": b, "flops": fl}
    counts, _ = _per_seq(case)
    m, m_out = sum(n for n, _ in counts), sum(k for _, k in counts)
    n_layers = case.get("layers", 1)
    b0, f0 = layer(m, m_out, False)
    b1, f1 = layer(m_out, m_out, False)
    total_b, total_f = b0 + (n_layers - 1) * b1, f0 + (n_layers - 1) * f1
    if case["kind"] == "loop":
        total_b, total_f = 4 * n_layers * b1, 4 * n_layers * f1
        if case["approx"]:
            # q, scores and the context update of every other token of the step (all, then three times the
            # response); the values that changed are those of the candidates
            toks = T + 3 * B * min(RESP, L // 2) - 4 * m
            keys = (m / B) if case["approx"] == 2 else L
            total_f += n_layers * toks * (2.0 * d * dq + 2.0 * keys * dq + 2.0 * (m / B) * dq)
            total_b += n_layers * toks * float(d + 2 * dq) * e
    return {"bytes": total_b, "flops": total_f}


def tolerance(case):
    # Measured with the sums in another order (other tiles and key splits): bf16 layers differ by 1e-3, and a
    # stack carries that from layer to layer; fp32 sums have at most a few thousand terms.  The lists and
    # flags are whole numbers, and no cosine lies near tau.
    if SHAPES[case["shape"]].dtype == "f32" or case["kind"] == "saliency":
        return {"rel": 1e-5, "differ": 0.0}
    return {"rel": 4e-3 if case.get("layers", 1) == 1 else 1e-2, "differ": 0.0}
