"""Performance cases: the calls a serving program makes, over the sizes it makes them at.

A case names a call (``prefill``: the shared-stage forward; ``decode``: the
downstream step; ``graph``: the same step replayed from a captured graph;
``dit``: the denoising step), a layer shape of ``workloads``, the compute-unit
budget, the weight format, the key/value placement and the ranges its sequence
lengths are drawn from.  The lengths follow from the case alone
(``shape_seed``), every value from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2608_01785_amd import binding, device_data
from paper_2608_01785_amd import workloads as wl

SHAPES = {"tiny": wl.TINY, "thinker": wl.THINKER, "talker": wl.TALKER, "mixed": wl.THINKER_MIXED, "dit": wl.DIT}
LADDER = (64, 96, 128, 160, 192, 256)   # a context's ladder; its complements are 192 .. 64
SECTIONS = {64: (8, 12, 12), 128: (16, 24, 24)}


def _case(name, call, model, layers, cus, **more):
    c = dict(name=name, call=call, model=model, layers=layers, cus=cus, weights="f16", seqs=1, lo=1, hi=1,
             ctx_lo=0, ctx_hi=0, singles=0, single_lo=0, single_hi=0, cache="none", page=0, bias=False,
             mrope=False, chunked=False, shape_seed=1)
    c.update(more)
    return c


def listed():
    return [
        # The smallest call: one small layer over two short requests, weights as they come (bf16).
        _case("tiny_prefill", "prefill", "tiny", 1, 64, weights="bf16", seqs=2, lo=96, hi=128),
        # The headline: eight requests of 256-2048 rows through four layers on the whole chip.
        _case("thinker_prefill", "prefill", "thinker", 4, 256, seqs=8, lo=256, hi=2048, shape_seed=12),
        # One scheduling step of the serving loop: an FCFS batch of a few requests, cache built, part of the chip.
        _case("thinker_batch", "prefill", "thinker", 1, 192, seqs=5, lo=256, hi=1024, cache="slots", shape_seed=3),
        # A single short multimodal request (image rows, then text), the latency a short-path request sees.
        _case("thinker_request", "prefill", "thinker", 1, 160, seqs=1, lo=389, hi=389, cache="slots", bias=True,
              mrope=True),
        # Chunked prefill and decode rows in one step beside a downstream stage.
        _case("mixed_step", "prefill", "mixed", 1, 96, seqs=4, lo=2048, hi=2048, chunked=True, singles=64,
              single_lo=4096, single_hi=4096, cache="slots", shape_seed=5),
        # Ragged ends of long prompts: short chunks behind long cached prefixes in a paged cache, bf16 weights.
        _case("paged_chunks", "prefill", "mixed", 1, 128, weights="bf16", seqs=3, lo=40, hi=300, ctx_lo=1000,
              ctx_hi=4000, singles=9, single_lo=100, single_hi=3000, cache="pages", page=256, shape_seed=7),
        # The downstream model's own prompts: the small dense layer, several short requests.
        _case("talker_prefill", "prefill", "talker", 4, 128, seqs=6, lo=40, hi=400, cache="slots", shape_seed=4),
        # The downstream decode step on half the chip.
        _case("talker_decode", "decode", "talker", 16, 128, seqs=32, ctx_lo=128, ctx_hi=1024, cache="slots"),
        # The same at a full batch, replayed from a captured graph.
        _case("talker_graph", "graph", "talker", 16, 160, seqs=128, ctx_lo=128, ctx_hi=1024, cache="slots"),
        # The shared stage's own decode: a few rows behind medium prompts, all compute units.
        _case("thinker_decode", "prefill", "thinker", 4, 256, singles=16, seqs=0, single_lo=1024, single_hi=2048,
              cache="slots", shape_seed=2),
        # A denoising step of four 32 x 32 latents on half the chip.
        _case("dit_step", "dit", "dit", 16, 128, seqs=4, lo=1024, hi=1024),
        # A few blocks over small ragged latents on a quarter of the chip, bf16 weights.
        _case("dit_ragged", "dit", "dit", 4, 64, weights="bf16", seqs=3, lo=77, hi=520, shape_seed=9),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes over their logarithm, every budget, format and placement."""
    call = rng.choice(("prefill", "prefill", "prefill", "decode", "graph", "dit"))
    cus = rng.choice(LADDER)
    down = min(cus, 192)                     # the downstream side never has the whole chip
    more = dict(weights=rng.choice(("f16", "f16", "bf16")), shape_seed=rng.randrange(1 << 20))
    if call == "dit":
        rows, n = _log(rng, 64, 4096), rng.randint(1, 6)
        hi = max(8, min(1024, rows // n))
        c = _case("", call, "dit", rng.randint(1, 8), down, seqs=n, lo=max(1, hi // rng.randint(1, 4)), hi=hi, **more)
    elif call in ("decode", "graph"):
        model = rng.choice(("talker", "talker", "thinker"))
        layers = rng.randint(4, 16) if model == "talker" else rng.randint(1, 3)
        hi = _log(rng, 64, 2048)
        page = rng.choice((0, 0, 64, 256, 1024))
        c = _case("", call, model, layers, down, seqs=min(_log(rng, 1, 200), 131072 // hi), ctx_lo=hi // 8, ctx_hi=hi,
                  cache="pages" if page else "slots", page=page, **more)
    else:
        model = rng.choice(("thinker", "mixed", "talker", "tiny"))
        rows, n = _log(rng, 24, 4096 if model == "talker" else 8192), rng.randint(1, 8)
        hi = max(2, min(2048, rows // n))
        cache = rng.choice(("none", "slots", "pages"))
        if cache != "none":
            more.update(ctx_hi=rng.choice((0, _log(rng, 64, 4096))), singles=rng.choice((0, _log(rng, 1, 48))),
                        single_lo=64, single_hi=_log(rng, 64, 4096),
                        page=rng.choice((64, 128, 512)) if cache == "pages" else 0)
        most = 4 if model in ("talker", "tiny") else 2 if rows < 4096 else 1
        c = _case("", call, model, rng.randint(1, most), cus, seqs=n, lo=max(2, hi // rng.randint(1, 8)), hi=hi,
                  cache=cache, bias=rng.random() < 0.3, mrope=rng.random() < 0.3, **more)
    del c["name"]
    return c


# ---------------------------------------------------------------------------- shapes

def _lengths(case):
    """(new rows, cached rows) of every sequence."""
    r = random.Random(case["shape_seed"])
    if case["call"] in ("decode", "graph"):
        return [1] * case["seqs"], [r.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(case["seqs"])]
    lens = [r.randint(case["lo"], case["hi"]) for _ in range(case["seqs"])]
    ctx = [r.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(case["seqs"])]
    if case["chunked"]:   # whole chunks behind 0, 1, 2, ... earlier chunks of their prompts
        ctx = [case["hi"] * i for i in range(case["seqs"])]
    lens += [1] * case["singles"]
    ctx += [r.randint(case["single_lo"], case["single_hi"]) for _ in range(case["singles"])]
    return lens, ctx


def _shape(case):
    s = SHAPES[case["model"]]
    if case["call"] == "dit":
        return s
    sec = SECTIONS[s.head_dim] if case["mrope"] else (0, 0, 0)
    return wl.LayerShape(s.hidden, s.n_q_heads, s.n_kv_heads, s.head_dim, s.ffn, s.rms_eps, s.rope_base, sec)


def _positions(case, lens, ctx):
    """[3, T] row positions: 1-D, or an image of half the rows followed by text."""
    if case["mrope"]:
        return wl.mrope_positions(lens, [n // 2 for n in lens], ctx, grid_w=16)
    p = np.concatenate([c + np.arange(n) for n, c in zip(lens, ctx)]).astype(np.int32)
    return np.stack([p, p, p])


def work(case):
    lens, ctx = _lengths(case)
    s, T, L = _shape(case), sum(lens), case["layers"]
    if case["call"] == "dit":
        d = s.hidden
        pairs = sum(n * n for n in lens)
        ada = 6 * d * d
        return {"bytes": L * 2 * (s.params_per_layer + 13 * d) + 6 * T * d + 4 * len(lens) * d,
                "flops": L * (2 * T * (s.params_per_layer - ada) + 2 * len(lens) * ada + 4 * d * pairs)}
    pairs = sum(n * c + n * (n + 1) // 2 for n, c in zip(lens, ctx))
    kv = s.n_kv_heads * s.head_dim * 4           # fp16 key and value bytes of one position
    cached = case["cache"] != "none"
    return {"bytes": L * (2 * s.params_per_layer + (kv * (sum(ctx) + T) if cached else 0)) + 6 * T * s.hidden,
            "flops": L * (2 * T * s.params_per_layer + 4 * s.n_q_heads * s.head_dim * pairs)}


def tolerance(case):
    # fp16 operands (2^-11 per rounding, independent errors) with fp32 sums and an fp32 residual
    # stream.  Largest distance from float64 over the listed and drawn cases: thinker 7.7e-4 (four
    # layers), mixed 3.6e-4, talker 4.2e-4 (sixteen), dit 2.2e-4 (sixteen), tiny 3.6e-5.
    rel = {"thinker": 3e-3, "mixed": 1.5e-3, "talker": 1.7e-3, "dit": 9e-4, "tiny": 1.5e-4}[case["model"]]
    return {"rel": rel, "max": 10 * rel}


# ---------------------------------------------------------------------------- inputs

_context = None


def _ctx():
    """The program's one context: its ladder of streams is built once."""
    global _context
    if _context is None:
        _context = binding.hs_context_create(0, LADDER)
    return _context


def _rand(gen, shape, std=1.0, dtype=torch.bfloat16, mean=0.0):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).add_(mean).to(dtype)


def _inputs(case, seed):
    """Weights, rows and cache contents, drawn on the GPU from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s, (lens, ctx) = _shape(case), _lengths(case)
    T, L = sum(lens), case["layers"]
    if case["call"] == "dit":
        shapes = wl.dit_weight_shapes(s)
        w = [{n: _rand(gen, shp, 0.02) for n, shp in shapes.items()} for _ in range(L)]
        return dict(w=w, x=_rand(gen, (T, s.hidden)), cond=_rand(gen, (len(lens), s.hidden), dtype=torch.float32))
    w = []
    for _ in range(L):
        lw = {n: _rand(gen, shp, 0.02, mean=1.0 if n.startswith("ln") else 0.0)
              for n, shp in wl.weight_shapes(s).items()}
        if case["bias"]:
            lw["b_qkv"] = _rand(gen, (s.qkv_rows,), 0.1)
        w.append(lw)
    got = dict(w=w, x=_rand(gen, (T, s.hidden)))
    if case["cache"] != "none":
        need = max(n + c for n, c in zip(lens, ctx)) + 1
        if case["cache"] == "pages":
            page = case["page"]
            pps = -(-need // page)
            perm = np.random.RandomState(seed % (1 << 31)).permutation(len(lens) * pps).astype(np.int32)
            got["table"], slots, span = perm.reshape(len(lens), pps), len(lens) * pps, page
        else:
            got["table"], slots, span = None, len(lens), -(-need // 64) * 64
        k = torch.empty((L, slots, s.n_kv_heads, span, s.head_dim), dtype=torch.float16, device="cuda")
        v = torch.empty((L, slots, s.n_kv_heads, span // 32, s.head_dim, 32), dtype=torch.float16, device="cuda")
        for t in (k, v):
            for l in range(L):
                t[l].normal_(generator=gen)
        got.update(k=k, v=v, slots=slots, span=span)
    return got


def prepare(case, seed):
    ctx = _ctx()
    s, (lens, cached) = _shape(case), _lengths(case)
    st = _inputs(case, seed)
    T, B = sum(lens), len(lens)
    st.update(ctx=ctx, call=case["call"], shape=s, lens=lens, cached=cached, cus=case["cus"],
              off=np.concatenate([[0], np.cumsum(lens)]).astype(np.int32),
              out=torch.zeros((T, s.hidden), dtype=torch.float32, device="cuda"))
    torch.cuda.synchronize()
    raw = st["w"]
    if case["weights"] == "f16":
        st["w"] = (device_data.prepare_dit_f16 if case["call"] == "dit" else device_data.prepare_f16)(ctx, raw)
    st["pos3"] = _positions(case, lens, cached) if case["mrope"] else None
    if case["call"] == "dit":
        st["ws"] = torch.empty(binding.hs_dit_workspace_size(s, T, B), dtype=torch.uint8, device="cuda")
        return st
    kv = None
    if "k" in st:
        kv = (list(st["k"]), list(st["v"]), st["slots"], st["span"])
        if st["table"] is not None:
            kv += (st["table"],)
    st["kv"] = kv
    top = max(n + c for n, c in zip(lens, cached)) + 1
    if case["call"] == "graph":
        top = st["table"].shape[1] * st["span"] if st["table"] is not None else st["span"]
    size = binding.hs_workspace_size_paged(s, T, B, top, case["page"] if case["cache"] == "pages" else 0)
    st["ws"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    if case["call"] == "graph":
        st["graph"] = binding.DecodeGraph(ctx, s, st["w"], st["x"], st["out"], kv, B, case["cus"], workspace=st["ws"])
    return st


def run(st):
    a = (st["ctx"], st["shape"], st["w"], st["x"], st["out"])
    if st["call"] == "dit":
        binding.hs_dit_forward(*a, st["cond"], st["off"], st["cus"], workspace=st["ws"])
        return {"x": st["out"]}
    if st["call"] == "graph":
        st["graph"].launch(st["cached"], st["table"])
    elif st["call"] == "decode":
        binding.hs_downstream_decode_step(*a, st["kv"], st["cached"], st["cus"], workspace=st["ws"])
    elif st["pos3"] is not None:
        binding.hs_shared_stage_forward_mrope(*a, st["off"], st["pos3"], ctx_lens=st["cached"] if st["kv"] else None,
                                              kv=st["kv"], cu_budget=st["cus"], workspace=st["ws"])
    else:
        binding.hs_shared_stage_forward(*a, st["off"], ctx_lens=st["cached"] if st["kv"] else None, kv=st["kv"],
                                        cu_budget=st["cus"], workspace=st["ws"])
    return {"x": st["out"], "k": st["k"], "v": st["v"]} if st["kv"] else {"x": st["out"]}


# ---------------------------------------------------------------------------- float64

def _rope64(x, pos3, base, sections):
    """x [T, H, dh]; pairs (j, j + dh/2) turn by the position of their section."""
    half = x.shape[-1] // 2
    j = torch.arange(half, dtype=torch.float64, device=x.device)
    comp = torch.repeat_interleave(torch.arange(3, device=x.device), torch.tensor(sections, device=x.device))
    th = (pos3[comp].T * torch.pow(torch.tensor(base, dtype=torch.float64, device=x.device), -j / half))[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * th.cos() - b * th.sin(), b * th.cos() + a * th.sin()], -1)


def _attend64(q, k, v, first):
    """q [n, Hq, dh] at positions first .., k and v [m, Hkv, dh]; first None: every key is seen."""
    n, hq, dh = q.shape
    g = hq // k.shape[1]
    if n == 1:
        kk, vv = k.repeat_interleave(g, 1), v.repeat_interleave(g, 1)
        p = torch.softmax((kk * q).sum(-1) / math.sqrt(dh), 0)
        return (p[..., None] * vv).sum(0)[None]
    out = torch.empty_like(q)
    for h in range(hq):
        sc = q[:, h] @ k[:, h // g].T.contiguous() / math.sqrt(dh)
        if first is not None:
            hide = torch.arange(k.shape[0], device=q.device)[None] > first + torch.arange(n, device=q.device)[:, None]
            sc.masked_fill_(hide, -math.inf)
        out[:, h] = torch.softmax(sc, -1) @ v[:, h // g]
    return out


def _exact_dit(case, got, lens):
    s, x, c = _shape(case), got["x"].double(), got["cond"].double()
    d, H, dh = s.hidden, s.n_heads, s.head_dim
    seq = torch.repeat_interleave(torch.arange(len(lens), device="cuda"), torch.tensor(lens, device="cuda"))

    def norm(t):
        m = t.mean(-1, keepdim=True)
        return (t - m) / torch.sqrt(((t - m) ** 2).mean(-1, keepdim=True) + s.ln_eps)

    for lw in got["w"]:
        w = {n: t.double() for n, t in lw.items()}
        mod = ((c * torch.sigmoid(c)) @ w["w_ada"].T + w["b_ada"]).reshape(-1, 6, d)[seq]
        q, k, v = ((norm(x) * (1 + mod[:, 1]) + mod[:, 0]) @ w["w_qkv"].T + w["b_qkv"]).reshape(-1, 3, H, dh).unbind(1)
        o = torch.cat([_attend64(a, b, e, None) for a, b, e in zip(q.split(lens), k.split(lens), v.split(lens))])
        x = x + mod[:, 2] * (o.reshape(-1, d) @ w["w_o"].T + w["b_o"])
        z = (norm(x) * (1 + mod[:, 4]) + mod[:, 3]) @ w["w_fc1"].T + w["b_fc1"]
        a = 0.5 * z * (1 + torch.tanh(math.sqrt(2 / math.pi) * (z + 0.044715 * z ** 3)))
        x = x + mod[:, 5] * (a @ w["w_fc2"].T + w["b_fc2"])
    return {"x": x}


def exact(case, seed):
    lens, ctx = _lengths(case)
    got = _inputs(case, seed)
    if case["call"] == "dit":
        return _exact_dit(case, got, lens)
    s, x, T = _shape(case), got["x"].double(), sum(lens)
    hq, hkv, dh, f = s.n_q_heads, s.n_kv_heads, s.head_dim, s.ffn
    pos3 = torch.from_numpy(_positions(case, lens, ctx)).to("cuda", torch.float64)
    sections = s.mrope_sections if any(s.mrope_sections) else (dh // 2, 0, 0)
    cache = "k" in got
    k_all = v_all = None
    if cache:
        k_all, v_all = got["k"].double(), got["v"].double()
    span = got.get("span", 1)

    def norm(t, g):
        return t / torch.sqrt((t * t).mean(-1, keepdim=True) + s.rms_eps) * g

    for l, lw in enumerate(got["w"]):
        w = {n: t.double() for n, t in lw.items()}
        qkv = norm(x, w["ln1"]) @ w["w_qkv"].T
        if "b_qkv" in w:
            qkv = qkv + w["b_qkv"]
        q, k, v = (t.reshape(T, -1, dh) for t in qkv.split([hq * dh, hkv * dh, hkv * dh], 1))
        q, k = _rope64(q, pos3, s.rope_base, sections), _rope64(k, pos3, s.rope_base, sections)
        o, t0 = [], 0
        for b, (n, c) in enumerate(zip(lens, ctx)):
            kb, vb, qb = k[t0:t0 + n], v[t0:t0 + n], q[t0:t0 + n]
            t0 += n
            if cache:
                p = np.arange(c + n)
                slot = np.full(c + n, b) if got["table"] is None else got["table"][b, p // span]
                sl, i = torch.from_numpy(slot).to("cuda", torch.int64), torch.from_numpy(p % span).to("cuda")
                k_all[l][sl[c:], :, i[c:]] = kb
                v_all[l][sl[c:], :, i[c:] // 32, :, i[c:] % 32] = vb
                kb, vb = k_all[l][sl, :, i], v_all[l][sl, :, i // 32, :, i % 32]
            o.append(_attend64(qb, kb, vb, c))
        h = x + torch.cat(o).reshape(T, -1) @ w["w_o"].T
        gu = norm(h, w["ln2"]) @ w["w_gate_up"].T
        x = h + (gu[:, :f] * torch.sigmoid(gu[:, :f]) * gu[:, f:]) @ w["w_down"].T
    return {"x": x, "k": k_all, "v": v_all} if cache else {"x": x}
