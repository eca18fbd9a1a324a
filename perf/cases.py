"""The work a user of this library has it do, as cases that can be timed and checked.

A case is one call (a training case: the forward and the backward of one layer) through the public
entry points. The listed cases are the repository's own configurations and the calls around them that
a model with sparsified layers makes: decode steps for one user and for a full batch, decode inside a
paged serving engine, verification of a few speculated tokens, chunked and whole-prompt prefill, a
training step, and the small fp32 prefill; ``draw`` gives more of the same ranges. Inputs are iid
N(0, 1) rounded to the case's type, as everywhere in this repository.
"""
import math

import numpy as np
import torch

import paper_2512_23966_amd as loza

DEV = "cuda"
MLA = {"Hq": 64, "Hkv": 1, "d_qk": 576, "d_v": 512, "shared": True, "scale": 192 ** -0.5}
D128 = {"Hq": 32, "d_qk": 128, "d_v": 128, "shared": False, "scale": 128 ** -0.5}
# token-granular: sink tokens, window tokens; block-granular (block > 0): sink blocks, local blocks
LONG = {"sink": 128, "window": 8192, "block": 0}     # the 128K / 1M configurations
SHORT = {"sink": 128, "window": 4096, "block": 0}    # the 32K multi-head configuration
PAPER = {"sink": 1, "window": 7, "block": 128}       # 1 sink block + 7 local blocks of 128 tokens


def listed():
    return [
        # one user's next token on a long context: launches and latency
        {"name": "decode_mla_b1", "op": "decode", "B": 1, "S_max": 131072, "len_lo": 65536, "page": 0, **MLA, **LONG},
        # the decode configuration: a full batch on caches of 64K to 256K rows
        {"name": "decode_mla_b64", "op": "decode", "B": 64, "S_max": 262144, "len_lo": 65536, "page": 0, **MLA, **LONG},
        # a serving engine's step with the paper's pattern, pages scattered over the pool, a batch of odd size
        {"name": "decode_mla_paged_paper_b43", "op": "decode", "B": 43, "S_max": 65536, "len_lo": 4096, "page": 128, **MLA, **PAPER},
        # grouped heads of width 128 (4 query heads on a key head), caches of odd length
        {"name": "decode_gqa128_b16", "op": "decode", "B": 16, "S_max": 32749, "len_lo": 8192, "page": 0, "Hkv": 8, **D128, **SHORT},
        # verification of 4 speculated tokens for 16 sequences of a paged engine
        {"name": "extend_mla_paged_q4_b16", "op": "extend", "q_len": 4, "B": 16, "S_max": 65536, "len_lo": 16384, "page": 128, **MLA, **LONG},
        # chunked prefill: 4 sequences take 1000 more tokens (not a multiple of any tile)
        {"name": "extend_mla_q1000_b4", "op": "extend", "q_len": 1000, "B": 4, "S_max": 65536, "len_lo": 16384, "page": 0, **MLA, **LONG},
        # whole-prompt prefill with the paper's pattern at the shortest context it trains
        {"name": "prefill_mla_paper_32k", "op": "prefill", "dtype": "bf16", "B": 1, "S": 32768, **MLA, **PAPER},
        # the headline prefill: 128K tokens, sink 128, window 8192
        {"name": "prefill_mla_128k", "op": "prefill", "dtype": "bf16", "B": 1, "S": 131072, **MLA, **LONG},
        # the multi-head configuration (32 heads of width 128, 32K tokens)
        {"name": "prefill_mha128_32k", "op": "prefill", "dtype": "bf16", "B": 1, "S": 32768, "Hkv": 32, **D128, **SHORT},
        # the fp32 configuration: one head, 1024 tokens
        {"name": "prefill_f32_1k", "op": "prefill", "dtype": "f32", "B": 1, "S": 1024, "Hq": 1, "Hkv": 1, "d_qk": 64, "d_v": 64,
         "shared": False, "scale": 64 ** -0.5, "sink": 64, "window": 256, "block": 0},
        # a training step of a sparsified layer (forward and gradients) with the paper's pattern
        {"name": "train_mla_paper_16k", "op": "train", "dtype": "bf16", "B": 1, "S": 16384, **MLA, **PAPER},
        # the same for heads of width 128, ragged length
        {"name": "train_mha128_8k", "op": "train", "dtype": "bf16", "B": 1, "S": 8111, "Hkv": 32, **D128, **SHORT},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("decode", "decode", "extend", "prefill", "prefill", "train", "f32"))
    if op == "f32":
        d = rng.choice((64, 96, 128))
        return {"op": "prefill", "dtype": "f32", "B": 1, "S": _log(rng, 256, 2048), "Hq": rng.choice((1, 2, 4)), "Hkv": 1, "d_qk": d, "d_v": d,
                "shared": False, "scale": d ** -0.5, "sink": rng.choice((0, 16, 64)), "window": _log(rng, 64, 512), "block": 0}
    wide = rng.random() < 0.65
    head = dict(MLA) if wide else {"Hkv": rng.choice((8, 32)), **D128}
    pat = dict(rng.choice((LONG, PAPER)) if wide else rng.choice((SHORT, PAPER)))
    if op == "decode":
        s = _log(rng, 4096, 262144 if wide else 65536)
        page = rng.choice((0, 64, 128))
        if page:
            s = (s + page - 1) // page * page
        return {"op": op, "B": _log(rng, 1, 64 if wide else 32), "S_max": s, "len_lo": max(1, s // rng.choice((2, 4, 16))), "page": page, **head, **pat}
    if op == "extend":
        s = _log(rng, 8192, 65536)
        page = rng.choice((0, 128))
        if page:
            s = (s + page - 1) // page * page
        return {"op": op, "q_len": _log(rng, 2, 2048), "B": _log(rng, 1, 16), "S_max": s, "len_lo": s // 2, "page": page, **head, **pat}
    if op == "prefill":
        return {"op": op, "dtype": "bf16", "B": 1, "S": _log(rng, 512, 65536 if wide else 32768), **head, **pat}
    return {"op": "train", "dtype": "bf16", "B": 1, "S": _log(rng, 768, 16384 if wide else 8192), **head, **pat}


# ---- inputs ------------------------------------------------------------------------------------------

def _normal(gen, dtype, *shape):
    t = torch.empty(shape, dtype=dtype, device=DEV)
    flat = t.view(-1)
    step = 1 << 28
    for a in range(0, flat.numel(), step):
        b = min(flat.numel(), a + step)
        flat[a:b].copy_(torch.randn(b - a, generator=gen, device=DEV, dtype=torch.float32))
    return t


def _inputs(case, seed):
    """The tensors a program holds before the call, from the seed alone."""
    c = case
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    if c["op"] in ("prefill", "train"):
        dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
        s = {"q": _normal(gen, dt, c["B"], c["S"], c["Hq"], c["d_qk"]), "k": _normal(gen, dt, c["B"], c["S"], c["Hkv"], c["d_qk"])}
        s["v"] = s["k"] if c["shared"] else _normal(gen, dt, c["B"], c["S"], c["Hkv"], c["d_v"])
        if c["op"] == "train":
            s["dout"] = _normal(gen, dt, c["B"], c["S"], c["Hq"], c["d_v"])
        return s
    bf = torch.bfloat16
    lens = rng.integers(c["len_lo"], c["S_max"] + 1, size=c["B"]).astype(np.int32)
    if c["op"] == "extend":
        lens = np.maximum(lens, min(c["q_len"], c["S_max"])).astype(np.int32)
        s = {"q": _normal(gen, bf, c["B"], c["q_len"], c["Hq"], c["d_qk"])}
    else:
        s = {"q": _normal(gen, bf, c["B"], c["Hq"], c["d_qk"])}
    if c["page"]:
        per = c["S_max"] // c["page"]
        rows = (c["B"] * per, c["page"])
        s["table"] = torch.from_numpy(rng.permutation(c["B"] * per).astype(np.int32).reshape(c["B"], per)).to(DEV)
    else:
        rows = (c["B"], c["S_max"])
    s["k"] = _normal(gen, bf, *rows, c["Hkv"], c["d_qk"])
    s["v"] = s["k"] if c["shared"] else _normal(gen, bf, *rows, c["Hkv"], c["d_v"])
    s["lens_host"] = lens
    s["lens"] = torch.from_numpy(lens).to(DEV)
    return s


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["case"] = c
    lead = s["q"].shape[:-1]
    s["out"] = torch.empty(*lead, c["d_v"], dtype=s["q"].dtype, device=DEV)
    lse = (c["B"], c["Hq"]) if c["op"] == "decode" else (c["B"], c["Hq"], lead[1])
    s["lse"] = torch.empty(lse, dtype=torch.float32, device=DEV)
    mult = c["block"] or 1
    if c["op"] == "decode":
        n = loza.loza_ssa_decode_workspace_bytes(c["B"], c["Hq"], c["Hkv"], c["S_max"], c["d_v"], c["sink"] * mult, c["window"] * mult)
        s["ws"] = torch.empty(n, dtype=torch.uint8, device=DEV)
    if c["op"] == "train":
        s["dq"], s["dk"] = torch.empty_like(s["q"]), torch.empty_like(s["k"])
        s["dv"] = None if c["shared"] else torch.empty_like(s["v"])
        sizes = (c["B"], c["Hq"], c["Hkv"], c["S"], c["d_qk"], c["d_v"])
        if c["block"]:
            n = loza.loza_ssa_backward_workspace_bytes_blocks(*sizes, c["sink"], c["window"], c["block"], c["shared"])
        else:
            n = loza.loza_ssa_backward_workspace_bytes(*sizes, c["sink"], c["window"], c["shared"])
        s["ws"] = torch.empty(n, dtype=torch.uint8, device=DEV)
    return s


# ---- one pass ------------------------------------------------------------------------------------------

def run(s):
    c = s["case"]
    q, k, v, out, lse = s["q"], s["k"], s["v"], s["out"], s["lse"]
    pat = (c["sink"], c["window"], c["block"]) if c["block"] else (c["sink"], c["window"])
    if c["op"] == "decode":
        if c["page"]:
            fn = loza.loza_ssa_decode_paged_blocks if c["block"] else loza.loza_ssa_decode_paged
            fn(q, k, v, s["table"], s["lens"], out, lse, *pat, c["scale"], s["ws"])
        else:
            fn = loza.loza_ssa_decode_blocks if c["block"] else loza.loza_ssa_decode
            fn(q, k, v, s["lens"], out, lse, *pat, c["scale"], s["ws"])
    elif c["op"] == "extend":
        if c["page"]:
            fn = loza.loza_ssa_extend_paged_blocks if c["block"] else loza.loza_ssa_extend_paged
            fn(q, k, v, s["table"], s["lens"], out, lse, *pat, c["scale"])
        else:
            fn = loza.loza_ssa_extend_blocks if c["block"] else loza.loza_ssa_extend
            fn(q, k, v, s["lens"], out, lse, *pat, c["scale"])
    elif c["dtype"] == "f32":
        fn = loza.loza_ssa_prefill_blocks_f32 if c["block"] else loza.loza_ssa_prefill_f32
        fn(q, k, v, out, lse, *pat, c["scale"])
    else:
        fn = loza.loza_ssa_prefill_blocks if c["block"] else loza.loza_ssa_prefill
        fn(q, k, v, out, lse, *pat, c["scale"])
        if c["op"] == "train":
            fn = loza.loza_ssa_backward_blocks if c["block"] else loza.loza_ssa_backward
            fn(q, k, v, out, lse, s["dout"], s["dq"], s["dk"], s["dv"], *pat, c["scale"], s["ws"])
            return [out, lse, s["dq"], s["dk"]] + ([] if c["shared"] else [s["dv"]])
    return [out, lse]


# ---- what a pass cannot do without -----------------------------------------------------------------------

def _window_begin(c, i):
    """First key of the window of position i (an int or an integer tensor)."""
    if c["block"]:
        b = (i // c["block"] - c["window"] + 1) * c["block"]
    else:
        b = i - c["window"] + 1
    return b.clamp(min=0) if isinstance(b, torch.Tensor) else max(0, b)


def _sink_end(c):
    return c["sink"] * (c["block"] or 1)


def _live(c, i):
    wb = _window_begin(c, i)
    return min(_sink_end(c), wb) + i + 1 - wb


def work(case):
    c = case
    es = 4 if c.get("dtype") == "f32" else 2
    row = (c["d_qk"] if c["shared"] else c["d_qk"] + c["d_v"]) * es      # key and value row of one key head
    pair = 2 * (c["d_qk"] + c["d_v"])                                    # forward flops of a (query head, key) pair
    q_row = (c["d_qk"] + c["d_v"]) * es + 4                              # query in, result and log-sum-exp out
    if c["op"] in ("prefill", "train"):
        pairs = c["B"] * c["Hq"] * sum(_live(c, i) for i in range(c["S"]))
        rows, keys = c["B"] * c["S"] * c["Hq"], c["B"] * c["S"] * c["Hkv"]
        w = {"bytes": rows * q_row + keys * row, "flops": pairs * pair}
        if c["op"] == "train":   # + q, k, v, out, lse, dout read; dq, dk, dv written
            w["bytes"] += rows * (2 * c["d_qk"] + 2 * c["d_v"]) * es + rows * 4 + 2 * keys * row
            w["flops"] += pairs * 2 * (3 * c["d_qk"] + 2 * c["d_v"])
        return w
    n = 64                                                               # lengths are uniform in [len_lo, S_max]
    lens = [c["len_lo"] + (c["S_max"] - c["len_lo"]) * (2 * t + 1) // (2 * n) for t in range(n)]
    if c["op"] == "decode":
        live = sum(_live(c, x - 1) for x in lens) / n
        return {"bytes": c["B"] * (c["Hkv"] * live * row + c["Hq"] * q_row), "flops": c["B"] * c["Hq"] * live * pair}
    ql = c["q_len"]
    lens = [max(x, ql) for x in lens]
    union = pairs = 0
    for x in lens:
        wb = _window_begin(c, x - ql)
        union += min(_sink_end(c), wb) + x - wb
        step = max(1, ql // 16)
        at = range(x - ql, x, step)
        pairs += ql * sum(_live(c, i) for i in at) / len(at)
    return {"bytes": c["B"] * (c["Hkv"] * union / n * row + ql * c["Hq"] * q_row), "flops": c["B"] * c["Hq"] * pairs / n * pair}


def tolerance(case):
    # About four times the error measured against 64-bit arithmetic (relative 2-norm; largest difference
    # over the larger of the value and the rms): bf16 forward 1.7e-3 to 2.3e-3 and 0.03 (the rounding of
    # the result and of the softmax weights), gradients 2.4e-3 and 0.19, fp32 3.5e-7 and 3.7e-6.
    if case.get("dtype") == "f32":
        return {"rel": 1.5e-6, "max": 1.5e-5}
    if case["op"] == "train":
        return {"rel": 1e-2, "max": 0.75}
    return {"rel": 8e-3, "max": 0.1}


# ---- the same in 64 bits ---------------------------------------------------------------------------------

def _mask(c, i, j):
    i, j = i[:, None], j[None, :]
    return (j <= i) & ((j < _sink_end(c)) | (j >= _window_begin(c, i)))


def _chunk(c, q, kk, vv, i, j):
    """Queries q [n, H, d] at positions i against keys kk [m, d] / values vv at positions j: softmax parts in 64 bits."""
    n, h, d = q.shape
    s = (q.reshape(n * h, d) @ kk.T).view(n, h, -1) * c["scale"]
    s.masked_fill_(~_mask(c, i, j)[:, None, :], -math.inf)
    lse = torch.logsumexp(s, -1)
    p = s.sub_(lse[..., None]).exp_()
    return p, (p.view(n * h, -1) @ vv).view(n, h, -1), lse


def _keys_of(c, i0, i1):
    """Positions that the queries i0 .. i1 see between them."""
    wb, se = _window_begin(c, i0), min(_sink_end(c), i1 + 1)
    return torch.cat([torch.arange(0, min(se, wb), device=DEV), torch.arange(wb, i1 + 1, device=DEV)])


def exact(case, seed):
    c = case
    if work(c)["flops"] > 4e13:
        return None
    s = _inputs(c, seed)
    f64, g_of = torch.float64, c["Hq"] // c["Hkv"]
    q = s["q"][:, None] if c["op"] == "decode" else s["q"]
    nb, nq = q.shape[:2]
    out = torch.empty(nb, nq, c["Hq"], c["d_v"], dtype=f64, device=DEV)
    lse = torch.empty(nb, c["Hq"], nq, dtype=f64, device=DEV)
    train = c["op"] == "train"
    if train:
        dq = torch.empty(q.shape, dtype=f64, device=DEV)
        dk = torch.zeros(s["k"].shape, dtype=f64, device=DEV)
        dv = torch.zeros(*s["k"].shape[:3], c["d_v"], dtype=f64, device=DEV)
    step = max(1, (512 if train else 1024) // max(1, g_of // 8))
    for b in range(nb):
        first = int(s["lens_host"][b]) - nq if "lens_host" in s else 0
        for a in range(0, nq, step):
            e = min(nq, a + step)
            i = torch.arange(first + a, first + e, device=DEV)
            j = _keys_of(c, first + a, first + e - 1)
            if c.get("page"):
                page = s["table"][b].long()[j // c["page"]]
                kr, vr = (s[n][page, j % c["page"]] for n in ("k", "v"))
            else:
                kr, vr = s["k"][b, j], s["v"][b, j]
            for g in range(c["Hkv"]):
                hs = slice(g * g_of, (g + 1) * g_of)
                qq, kk, vv = q[b, a:e, hs].to(f64), kr[:, g].to(f64), vr[:, g, : c["d_v"]].to(f64)
                p, o, ls = _chunk(c, qq, kk, vv, i, j)
                out[b, a:e, hs], lse[b, hs, a:e] = o, ls.T
                if train:
                    m, n = p.shape[-1], p.shape[0] * p.shape[1]
                    do = s["dout"][b, a:e, hs].to(f64)
                    p = p.view(n, m)
                    dv[b, :, g].index_add_(0, j, p.T @ do.reshape(n, -1))
                    dd = (do * o).sum(-1).reshape(n, 1)
                    ds = (do.reshape(n, -1) @ vv.T).sub_(dd).mul_(p).mul_(c["scale"])
                    dq[b, a:e, hs] = (ds @ kk).view(e - a, g_of, -1)
                    dk[b, :, g].index_add_(0, j, ds.T @ qq.reshape(n, -1))
    if c["op"] == "decode":
        return [out[:, 0], lse[:, :, 0]]
    if not train:
        return [out, lse]
    if c["shared"]:
        dk[..., : c["d_v"]] += dv
        return [out, lse, dq, dk]
    return [out, lse, dq, dk, dv]
