"""Performance cases of the spliced decode attention and of the decode loop around it.

Each case is one decode pass over one or more consecutive layers of a sweep, through the
public entry points of ``paper_2605_30574_amd``, with synthetic inputs of the shapes in
``workloads/configs.py`` (attention) and ``workloads/model.py`` (hidden sizes):

  attn     splice_decode_attn (or splice_decode_attn_noalloc), every cell at one step;
  step     splice_decode_step, every cell at its own step, the K/V row appended;
  forked   splice_decode_forked, cells that fork from the clean run at their onset;
  decode   decode.SweepDecoder.step, whole passes of a synthetic model.

``launch`` is "graph" where a program replays one captured graph of a step's layers (as
the benchmark does for a lock-step sweep) and "eager" where it calls the binding.
"""
from __future__ import annotations

import math
import random
import types

import numpy as np
import torch

import paper_2605_30574_amd as sp
from paper_2605_30574_amd import decode

DEV = "cuda"
SINK = 50.0             # sink outlier: prompt position 0, channels 0..3 of K

# attention shapes: (Hq, Hkv, D)
QWEN, GEMMA, TINY = (32, 8, 128), (8, 4, 256), (4, 2, 64)
# hidden sizes of the decode loop's models: (d_model, d_ff, vocabulary)
QWEN3_4B, LLAMA3_8B, QWEN3_8B = (2560, 9728, 151936), (4096, 14336, 128256), (4096, 12288, 151936)


def _attn(name, heads, **kw):
    c = dict(kind="attn", n_layers=36, first=18, layers=4, Hq=heads[0], Hkv=heads[1], D=heads[2], window=0, period=0,
             dtype="bf16", launch="graph", noalloc=False)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def _decode(name, model, **kw):
    c = dict(kind="decode", n_layers=2, layers=2, first=0, Hq=QWEN[0], Hkv=QWEN[1], D=QWEN[2], window=0, period=0,
             dtype="bf16", d_model=model[0], d_ff=model[1], vocab=model[2], weights="bf16", launch="eager")
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the tiny float32 sweep (two layers, six cells): the smallest calls, all latency and launches
        _attn("tiny-f32", TINY, n_layers=2, first=0, layers=2, cells=6, Tp=32, a=4, b=28, cap=16, step=9, donor="zero",
              dtype="f32", launch="eager"),
        # a handful of cells decoded interactively by a program that may not allocate: small calls, launched one by one
        _attn("few-cells-noalloc", QWEN, cells=5, Tp=256, a=40, b=236, cap=512, step=37, donor="blank", launch="eager",
              noalloc=True),
        # the Qwen3-4B-shaped sweep (80 cells, a 256-token prompt) in the middle of its decode
        _attn("qwen3-4b-sweep", QWEN, cells=80, Tp=256, a=40, b=236, cap=512, step=300, donor="blank"),
        # the Llama-3-8B-shaped sweep, ZERO donor: a 1024-token prompt whose span costs no bytes, an early step
        _attn("llama3-8b-zero", QWEN, n_layers=32, first=14, cells=64, Tp=1024, a=43, b=1003, cap=256, step=64,
              donor="zero"),
        # the Gemma-3-4B-shaped sweep: D = 256, five local layers (1024-key window) and a global one
        _attn("gemma3-4b-window", GEMMA, n_layers=34, first=12, layers=6, cells=48, Tp=4096, a=64, b=4064, cap=128,
              step=100, donor="blank", window=1024, period=6),
        # the Qwen3-8B-shaped long-context sweep at an early step: the shared 8192-token prompts, hardly any generated rows
        _attn("qwen3-8b-early", QWEN, cells=128, Tp=8192, a=128, b=8128, cap=1024, step=3, donor="diff"),
        # the same sweep near its end: half a gigabyte of generated rows a layer
        _attn("qwen3-8b-late", QWEN, cells=128, Tp=8192, a=128, b=8128, cap=1024, step=1000, donor="diff"),
        # continuous decoding of that sweep: cells at their own steps, some finished, K/V appended
        _attn("qwen3-8b-ragged", QWEN, kind="step", cells=128, Tp=8192, a=128, b=8128, cap=1024, step=1023, donor="diff",
              launch="eager"),
        # the Qwen3-4B-shaped sweep forked from one clean run, at a step where half the onsets have passed
        _attn("qwen3-4b-forked", QWEN, kind="forked", cells=80, Tp=256, a=40, b=236, cap=512, step=24, donor="blank"),
        # float32 caches (a precision control of a sweep): the Llama-3-8B shape, BLANK donor
        _attn("llama3-8b-f32", QWEN, n_layers=32, first=14, layers=2, cells=64, Tp=1024, a=43, b=1003, cap=256, step=128,
              donor="blank", dtype="f32", launch="eager"),
        # the greedy decode loop around a Qwen3-8B-sized model, a full batch of cells (two layers and the head)
        _decode("decode-qwen3-8b", QWEN3_8B, cells=128, Tp=1024, a=128, b=960, cap=256, step=255, donor="diff"),
        # the same loop around a Qwen3-4B-sized model with a few cells: weights streamed for hardly any rows
        _decode("decode-qwen3-4b-few", QWEN3_4B, cells=8, Tp=256, a=40, b=236, cap=128, step=127, donor="blank"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(("attn",) * 5 + ("step", "step", "forked", "decode", "decode"))
    donor = rng.choice(("blank", "diff", "zero"))
    while True:
        cells, Tp, cap = _log(rng, 2, 128), _log(rng, 16, 8192), _log(rng, 16, 1024)
        step = rng.randrange(cap)
        a = rng.randrange(0, max(1, Tp // 8))
        b = Tp - rng.randrange(0, max(1, Tp // 8))
        common = dict(cells=cells, Tp=Tp, a=a, b=b, cap=cap, step=step, donor=donor)
        if kind == "decode":
            c = _decode(None, rng.choice((QWEN3_4B, LLAMA3_8B, QWEN3_8B)), **dict(common, Tp=min(Tp, 2048), a=min(a, 200),
                        b=min(b, 2048), cap=min(cap, 256), step=step % 256 % min(cap, 256)))
            n = rng.choice((1, 2, 3))
            c.update(n_layers=n, layers=n)
        else:
            Hkv, G = rng.choice((1, 2, 4, 8)), rng.choice((1, 2, 4, 4, 8))
            f32 = kind == "attn" and rng.random() < 0.25
            c = _attn(None, (Hkv * G, Hkv, rng.choice((64, 128, 128, 256))), kind=kind, layers=rng.choice((1, 2, 4)), **common)
            c.update(window=rng.choice((0, 0, 1024, 300)), launch=rng.choice(("graph", "graph", "eager")))
            if f32:
                c.update(dtype="f32", cells=min(cells, 64), Tp=min(Tp, 2048), a=min(a, 200), b=min(b, 2048))
            elif kind == "attn" and rng.random() < 0.2:
                c.update(noalloc=True, launch="eager", cells=min(cells, 16))
        w, most = work(c), 250e9 if kind == "decode" else (70e9 if c["dtype"] == "bf16" else 2.4e9)
        if w["bytes"] < 2.25e9 and w["flops"] < most:
            return c


# ------------------------------------------------------------------------------------------------ inputs

def _cells(c):
    """(L, W) of every cell: onsets doubling from 0, cutoffs spread over the layers, never-spliced cells (L = N) among them."""
    Ws = (0, 1, 2, 4, 8, 16, 32, 64)
    lw = [(c["n_layers"] * ((i // len(Ws)) % 5) // 4, Ws[i % len(Ws)]) for i in range(c["cells"])]
    if c["cells"] > 1:
        lw[-1] = (c["n_layers"], 0)     # the clean run (a forked sweep's trunk)
    elif c["kind"] == "forked":
        lw[0] = (c["n_layers"], 0)
    return np.ascontiguousarray(np.array(lw, dtype=np.int32))


def _steps(c, seed):
    """Every cell's own step: uniform over the decode, the first and the last step present; of the attention's cells an
    eighth is finished (the decode loop's freed slots have been refilled: every row of its logits is a cell's)."""
    rng = np.random.default_rng([seed, 7])
    st = rng.integers(0, c["step"] + 1, size=c["cells"]).astype(np.int32)
    if c["kind"] == "step":
        st[rng.random(c["cells"]) < 0.125] = -1
    st[0] = c["step"]
    if c["cells"] > 1:
        st[-1] = 0
    return np.ascontiguousarray(st)


def _window(c, layer):
    return 0 if c["period"] and layer % c["period"] == c["period"] - 1 else c["window"]


def _inputs(c, seed):
    """The tensors of a pass: per layer the prompt caches (clean, donor), the generated caches, q and the new rows."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + 17)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def rn(*shape, std=1.0, dtype=dt):
        x = torch.randn(*shape, generator=g, device=DEV, dtype=dtype)
        return x.mul_(std) if std != 1.0 else x

    C, Hq, Hkv, D, Tp, cap = (c[k] for k in ("cells", "Hq", "Hkv", "D", "Tp", "cap"))
    layers = []
    for _ in range(c["layers"]):
        t = dict(clean_k=rn(Hkv, Tp, D), clean_v=rn(Hkv, Tp, D), donor_k=None, donor_v=None)
        t["clean_k"][:, 0, :4] *= SINK
        if c["donor"] != "zero":
            t["donor_k"], t["donor_v"] = rn(Hkv, Tp, D), rn(Hkv, Tp, D)
            t["donor_k"][:, 0, :4] *= SINK
            if c["donor"] == "blank":      # the scaffold around the span is kept
                for n in ("k", "v"):
                    t["donor_" + n][:, :c["a"]] = t["clean_" + n][:, :c["a"]]
                    t["donor_" + n][:, c["b"]:] = t["clean_" + n][:, c["b"]:]
        t["gen_k"], t["gen_v"] = rn(C, Hkv, cap, D), rn(C, Hkv, cap, D)
        if c["kind"] != "decode":
            t["q"] = rn(C, Hq, D)
        if c["kind"] == "step":
            t["k_new"], t["v_new"] = rn(C, Hkv, D), rn(C, Hkv, D)
        layers.append(t)
    s = dict(layers=layers)
    if c["kind"] == "decode":
        d, F, V = c["d_model"], c["d_ff"], c["vocab"]
        wdt = torch.bfloat16 if c["weights"] == "bf16" else torch.float32

        def wt(i, o, fan):
            return rn(i, o, std=fan ** -0.5, dtype=wdt)
        one = lambda: (1.0 + 0.1 * rn(d, dtype=torch.float32)).to(wdt)  # noqa: E731
        s["weights"] = dict(embed=wt(V, d, 1), lm_head=wt(d, V, d), norm_f=one(), layers=[
            dict(norm_1=one(), w_q=wt(d, Hq * D, d), w_k=wt(d, Hkv * D, d), w_v=wt(d, Hkv * D, d), w_o=wt(Hq * D, d, Hq * D),
                 norm_2=one(), w_gate=wt(d, F, d), w_up=wt(d, F, d), w_down=wt(F, d, F)) for _ in range(c["layers"])])
        s["tokens"] = torch.randint(0, V, (C,), generator=g, device=DEV)
    return s


def _shape(c):
    return sp.make_shape(c["cells"], c["n_layers"], c["Hq"], c["Hkv"], c["D"], c["Tp"], (c["a"], c["b"]), c["cap"],
                         c["donor"] == "zero", c["dtype"])


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["case"], s["lw"] = c, _cells(c)
    if c["kind"] in ("step", "decode"):
        s["steps"] = _steps(c, seed)
    if c["kind"] == "decode":
        w = types.SimpleNamespace(n_layers=c["n_layers"], n_q_heads=c["Hq"], n_kv_heads=c["Hkv"], head_dim=c["D"],
                                  prompt_len=c["Tp"], span=(c["a"], c["b"]), n_steps=c["cap"], donor=c["donor"],
                                  window=lambda layer: 0)
        m = types.SimpleNamespace(d_model=c["d_model"], d_ff=c["d_ff"], vocab=c["vocab"], eos=0, rope_theta=1.0e6,
                                  rms_eps=1.0e-6)
        s["decoder"] = decode.SweepDecoder(w, m, s["weights"], s["layers"], s["lw"], device=DEV)
        return s
    s["shape"] = _shape(c)
    s["calls"] = [sp.make_call(c["first"] + i, 0 if c["kind"] == "step" else c["step"], _window(c, c["first"] + i),
                               c["D"] ** -0.5) for i in range(c["layers"])]
    s["ws"] = None if c["noalloc"] else sp.new_workspace(s["shape"], device=DEV)
    s["out"] = [torch.zeros(c["cells"], c["Hq"], c["D"], device=DEV) for _ in s["calls"]]
    s["lse"] = [torch.zeros(c["cells"], c["Hq"], device=DEV) for _ in s["calls"]]
    if c["launch"] == "graph":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"], stream=side):
            _issue(s)
    return s


def _issue(s):
    c = s["case"]
    for i, call in enumerate(s["calls"]):
        t = s["layers"][i]
        prompt = (t["clean_k"], t["clean_v"], t["donor_k"], t["donor_v"], t["gen_k"], t["gen_v"], s["out"][i], s["lse"][i])
        if c["kind"] == "step":
            sp.splice_decode_step(s["shape"], call, s["lw"], s["steps"], t["q"], t["k_new"], t["v_new"], *prompt, s["ws"])
        elif c["kind"] == "forked":
            sp.splice_decode_forked(s["shape"], call, s["lw"], c["cells"] - 1, t["q"], *prompt, s["ws"])
        elif c["noalloc"]:
            sp.splice_decode_attn_noalloc(s["shape"], call, s["lw"], t["q"], *prompt)
        else:
            sp.splice_decode_attn(s["shape"], call, s["lw"], t["q"], *prompt, s["ws"])


def run(state):
    c = state["case"]
    if c["kind"] == "decode":
        tokens, logits = state["decoder"].step(state["tokens"], state["steps"])
        return {"tokens": tokens, "logits": logits, "gen_k": [t["gen_k"] for t in state["layers"]],
                "gen_v": [t["gen_v"] for t in state["layers"]]}
    if c["launch"] == "graph":
        state["graph"].replay()
    else:
        _issue(state)
    r = {"out": state["out"], "lse": state["lse"]}
    if c["kind"] == "step":
        r["gen_k"], r["gen_v"] = [t["gen_k"] for t in state["layers"]], [t["gen_v"] for t in state["layers"]]
    return r


# ------------------------------------------------------------------------------------------------ what a pass cannot do without

def _plan(c, seed=0):
    """Per layer: [(cell, step or -1, spliced, diverged)]."""
    lw = _cells(c)
    st = _steps(c, seed) if c["kind"] in ("step", "decode") else np.full(c["cells"], c["step"])
    for layer in range(c["first"], c["first"] + c["layers"]):
        yield layer, [(i, int(st[i]), bool(layer >= L and st[i] >= W), i == c["cells"] - 1 or
                       (L < c["n_layers"] and st[i] >= W)) for i, (L, W) in enumerate(lw.tolist())]


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    C, Hq, Hkv, D, Tp = (c[k] for k in ("cells", "Hq", "Hkv", "D", "Tp"))
    row = 2 * Hkv * D * e                                      # a K and a V row of every KV head
    nbytes = flops = 0
    for layer, cells in _plan(c):
        win = _window(c, layer)
        seen_clean, seen_donor, trunk_rows = np.zeros(Tp, bool), np.zeros(Tp, bool), 0
        for i, s, spl, div in cells:
            if s < 0 or (c["kind"] == "forked" and not div):
                continue
            j0 = Tp + s - win + 1 if win else 0
            jp, i0 = min(max(j0, 0), Tp), max(0, j0 - Tp)
            lo, hi = max(c["a"], jp), max(c["b"], jp)
            keys = Tp - jp + s + 1 - i0
            if spl:
                seen_clean[jp:lo] = True
                seen_clean[hi:] = True
                if c["donor"] != "zero":
                    seen_donor[lo:hi] = True
                else:
                    keys -= hi - lo
            else:
                seen_clean[jp:] = True
            own = s + 1 - i0
            if c["kind"] == "forked" and i != C - 1:            # rows below the onset are the trunk's
                own = max(0, s + 1 - max(i0, int(_cells(c)[i, 1])))
            nbytes += own * row + Hq * D * e
            if c["kind"] in ("step", "decode"):
                nbytes += row                                   # the new row is stored
            flops += 4 * keys * Hq * D
        nbytes += (int(seen_clean.sum()) + int(seen_donor.sum())) * row
        out = sum(1 for _, s, _, _ in cells if s >= 0)
        nbytes += out * Hq * (4 * D + 4)
    if c["kind"] == "decode":
        d, F, V = c["d_model"], c["d_ff"], c["vocab"]
        per = d * (Hq + 2 * Hkv) * D + Hq * D * d + 3 * d * F
        we = 2 if c["weights"] == "bf16" else 4
        nbytes += (per * c["layers"] + d * V) * we + C * d * we + C * V * 4
        flops += 2 * C * (per * c["layers"] + d * V)
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """Of a 64-bit pass, measured: 2e-4 to 4e-4 off in the bf16 attention (1.6e-3 at D = 256 with a window), 3e-7 in
    float32, 5e-3 to 8e-3 in a decode pass's logits, whose random head leaves near ties between tokens."""
    if case["kind"] == "decode":
        return {"rel": 2e-2, "differ": 0.5 if case["cells"] < 16 else 0.2}
    return {"rel": 6e-3} if case["dtype"] == "bf16" else {"rel": 1e-5}


# ------------------------------------------------------------------------------------------------ the same in 64 bits

def _attend64(c, layer, cells, t, q, lw, steps):
    """out, lse of every cell in 64 bits; a forked sweep's cells read the trunk's rows below their onset."""
    C, Hq, Hkv, D, Tp = (c[k] for k in ("cells", "Hq", "Hkv", "D", "Tp"))
    G, win, scale = Hq // Hkv, _window(c, layer), D ** -0.5
    out = torch.zeros(C, Hq, D, dtype=torch.float64, device=DEV)
    lse = torch.zeros(C, Hq, dtype=torch.float64, device=DEV)
    ck, cv = t["clean_k"].double(), t["clean_v"].double()
    dk, dv = (t["donor_k"].double(), t["donor_v"].double()) if t["donor_k"] is not None else (None, None)
    pos = torch.arange(Tp, device=DEV)
    span = (pos >= c["a"]) & (pos < c["b"])
    for i, s, spl, div in cells:
        if s < 0:
            continue
        j0 = Tp + s - win + 1 if win else 0
        jp, i0 = min(max(j0, 0), Tp), max(0, j0 - Tp)
        k, v = ck, cv
        if spl:
            m = span[None, :, None]
            zero = torch.zeros((), dtype=torch.float64, device=DEV)
            k, v = torch.where(m, zero if dk is None else dk, ck), torch.where(m, zero if dv is None else dv, cv)
        gk, gv = t["gen_k"][i, :, i0:s + 1].double(), t["gen_v"][i, :, i0:s + 1].double()
        if c["kind"] == "forked" and i != C - 1:
            n = max(0, min(int(lw[i][1]), s + 1) - i0)
            tk, tv = t["gen_k"][C - 1].double(), t["gen_v"][C - 1].double()
            gk, gv = torch.cat([tk[:, i0:i0 + n], gk[:, n:]], 1), torch.cat([tv[:, i0:i0 + n], gv[:, n:]], 1)
        keys, vals = torch.cat([k[:, jp:], gk], 1), torch.cat([v[:, jp:], gv], 1)      # [Hkv][n][D]
        sc = torch.bmm(q[i].view(Hkv, G, D), keys.transpose(1, 2).contiguous()) * scale
        l = torch.logsumexp(sc, -1)
        out[i] = torch.bmm(torch.exp(sc - l[..., None]), vals).view(Hq, D)
        lse[i] = l.view(Hq)
    return out, lse


def exact(case, seed):
    c = case
    s, lw = _inputs(c, seed), _cells(c).tolist()
    steps = _steps(c, seed)
    if c["kind"] == "decode":
        return _decode64(c, s, lw, steps)
    outs, lses = [], []
    for n, (layer, cells) in enumerate(_plan(c, seed)):
        t = s["layers"][n]
        if c["kind"] == "step":
            for i, st, _, _ in cells:
                if st >= 0:
                    t["gen_k"][i, :, st], t["gen_v"][i, :, st] = t["k_new"][i], t["v_new"][i]
        div = {i: d for i, _, _, d in cells}
        todo = [x for x in cells if c["kind"] != "forked" or div[x[0]]]
        o, l = _attend64(c, layer, todo, t, t["q"].double(), lw, steps)
        if c["kind"] == "forked":          # cells that have not diverged take the trunk's result
            for i in range(c["cells"]):
                if not div[i]:
                    o[i], l[i] = o[-1], l[-1]
        outs.append(o)
        lses.append(l)
    r = {"out": outs, "lse": lses}
    if c["kind"] == "step":
        r["gen_k"], r["gen_v"] = [t["gen_k"] for t in s["layers"]], [t["gen_v"] for t in s["layers"]]
    return r


def _decode64(c, s, lw, steps):
    """A pass of the decode loop in 64 bits, nothing rounded on the way but the caches' stored rows."""
    C, Hq, Hkv, D, Tp = (c[k] for k in ("cells", "Hq", "Hkv", "D", "Tp"))
    wt = s["weights"]
    p64 = Tp + torch.as_tensor(np.maximum(steps, 0), device=DEV).double()
    ang = p64[:, None] * (1.0e6 ** (-torch.arange(0, D // 2, device=DEV, dtype=torch.float64) * 2.0 / D))[None]
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def norm(x, g):
        return x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + 1.0e-6) * g.double()

    def rope(x):
        x1, x2 = x[..., :D // 2], x[..., D // 2:]
        return torch.cat([x1 * cos - x2 * sin, x2 * cos + x1 * sin], -1)

    def mul(h, w):     # in column blocks: a 64-bit copy of the head's weights would be large
        return torch.cat([h @ w[:, j:j + 16384].double() for j in range(0, w.shape[1], 16384)], -1)

    x = wt["embed"][s["tokens"]].double()
    for n, (layer, cells) in enumerate(_plan(c, 0)):
        p, t = wt["layers"][n], dict(s["layers"][n])
        cells = [(i, int(steps[i]), layer >= lw[i][0] and steps[i] >= lw[i][1], True) for i in range(C)]
        h = norm(x, p["norm_1"])
        q, k = rope(mul(h, p["w_q"]).view(C, Hq, D)), rope(mul(h, p["w_k"]).view(C, Hkv, D))
        v = mul(h, p["w_v"]).view(C, Hkv, D)
        t["gen_k"], t["gen_v"] = t["gen_k"].double(), t["gen_v"].double()
        for i, st, _, _ in cells:
            if st >= 0:
                t["gen_k"][i, :, st], t["gen_v"][i, :, st] = k[i], v[i]
        o, _ = _attend64(c, layer, cells, t, q, lw, steps)
        s["layers"][n] = t
        x = x + mul(o.view(C, Hq * D), p["w_o"])
        h = norm(x, p["norm_2"])
        gate = mul(h, p["w_gate"])
        x = x + mul(gate / (1.0 + torch.exp(-gate)) * mul(h, p["w_up"]), p["w_down"])
    logits = mul(norm(x, wt["norm_f"]), wt["lm_head"])
    return {"tokens": None, "logits": logits, "gen_k": [t["gen_k"] for t in s["layers"]],
            "gen_v": [t["gen_v"] for t in s["layers"]]}
