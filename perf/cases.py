"""Performance cases of the sparse prefill layer: the calls a program makes,
over the sizes it makes them at.

One pass of a layer case is what a prefill does per layer: estimation,
choices, permutations, block index and block-sparse attention for every head
(a plan is created from this layer's Q and K, executed and destroyed: the
pattern depends on the inputs, so no program keeps it for the next layer).
The other cases are the dense baseline through the same kernel, neighborhood
attention, the explicit row permutations and the offline pattern search.

`exact` is an independent statement of the path in plain torch at 64 bits:
token-pair predicates lifted to 64x64 blocks by brute force, a masked softmax
over the selected blocks.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2504_16083_amd import mmi
from synth import config as C
from synth import generate, search_space

DEV = "cuda" if torch.cuda.is_available() else "cpu"
D, B = 128, 64


# ------------------------------------------------------------------ the cases
def listed():
    def layer(name, family, S, Hq, Hkv, frame, texts, text, entry="plan", fused=False, lse=False):
        return {"name": name, "what": "layer", "family": family, "S": S, "Hq": Hq, "Hkv": Hkv, "frame": frame,
                "texts": texts, "text": text, "entry": entry, "fused": fused, "lse": lse}

    return [
        # one image-sized clip, a single pair of heads: launches and latency only
        layer("grid_4k", "grid", 4096, 2, 1, 252, 1, 64, entry="call"),
        # a short multi-turn prompt (two text turns, odd length) in a serving loop that may not allocate
        layer("short_3k", "modal", 3001, 28, 4, 196, 2, 200, entry="noalloc"),
        # a short video prompt: ragged length, Q/K/V as views of one fused projection, LSE asked for
        layer("clip_20k", "modal", 20240, 28, 4, 196, 3, 300, fused=True, lse=True),
        # 128 frames, Grid / A-shape / Vertical-Slash heads
        layer("video_32k", "mixed", 32768, 28, 4, 255, 1, 128),
        # a longer video, odd length, Q-Boundary heads with A-shape text and Grid video
        layer("video_66k", "qbgrid", 65800, 28, 4, 256, 2, 500),
        # text and video interleaved, all head kinds: the ordinary long prompt
        layer("mm_128k", "modal", 131072, 28, 4, 196, 4, 2304),
        # about 5% block density, attention sinks, eight KV heads
        layer("sinks_256k", "sinks", 262144, 32, 8, 256, 1, 256),
        # the benchmark's layer: 4088 frames and four text inserts
        layer("mm_1m", "long", 1048576, 28, 4, 256, 4, 512),
        # every causal block (the dense baseline; a model's dense layers), ragged, with LSE
        {"name": "dense_34k", "what": "dense", "S": 33950, "Hq": 28, "Hkv": 4, "lse": True},
        # one layer of a video DiT: bidirectional neighborhood attention over a token grid
        {"name": "natten_119k", "what": "natten", "T": 33, "H": 45, "W": 80, "wt": 9, "wh": 15, "ww": 15,
         "tt": 2, "th": 4, "tw": 8, "Hq": 24},
        # the Q/K/V gathers and the O scatter as explicit passes
        {"name": "permute_128k", "what": "permute", "S": 131072, "Hq": 28, "Hkv": 4, "frame": 196},
        # the offline pattern search on one calibration sample, the paper's search space
        {"name": "search_24k", "what": "search", "S": 24576, "Hq": 28, "Hkv": 4, "frame": 196, "texts": 2, "text": 1200},
    ]


def draw(rng: random.Random):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    what = rng.choice(["layer"] * 6 + ["dense", "natten", "permute", "search"])
    Hq, Hkv = rng.choice([(28, 4), (28, 4), (32, 8), (16, 2), (8, 8), (2, 1)])
    frame = rng.choice([196, 252, 255, 256, rng.randint(64, 400)])
    if what == "layer":
        S = size(1024, 262144)
        entry = rng.choice(["plan", "plan", "plan", "call"] + (["noalloc"] if S < 16384 else []))
        return {"what": what, "family": rng.choice(["grid", "mixed", "modal", "sinks", "long", "qbgrid"]), "S": S,
                "Hq": Hq, "Hkv": Hkv, "frame": frame, "texts": rng.randint(1, 5),
                "text": rng.randint(32, max(33, min(2048, S // 16))), "entry": entry, "fused": rng.random() < 0.3,
                "lse": rng.random() < 0.3}
    if what == "dense":
        return {"what": what, "S": size(1024, 65536), "Hq": Hq, "Hkv": Hkv, "lse": rng.random() < 0.5}
    if what == "natten":
        T, H, W = rng.choice([1, rng.randint(4, 24)]), rng.randint(24, 64), rng.randint(24, 72)
        odd = lambda n, hi: 2 * rng.randint(0, (min(n, hi) - 1) // 2) + 1  # noqa: E731
        tt, th, tw = (1, 8, 8) if T == 1 else rng.choice([(2, 4, 8), (4, 4, 4), (1, 8, 8)])
        return {"what": what, "T": T, "H": H, "W": W, "wt": odd(T, 9), "wh": odd(H, 21), "ww": odd(W, 21),
                "tt": tt, "th": th, "tw": tw, "Hq": rng.choice([8, 16, 24])}
    if what == "permute":
        return {"what": what, "S": size(4096, 262144), "Hq": Hq, "Hkv": Hkv, "frame": frame}
    return {"what": what, "S": size(2048, 12288), "Hq": Hq, "Hkv": Hkv, "frame": 196, "texts": 2,
            "text": rng.randint(64, 256)}


# ------------------------------------------------------------------ inputs
def layout(c):
    """Modality of every position: `texts` text runs (0) of `text` tokens, each
    followed by its share of the whole video frames (1); the rest of the
    tokens lengthen the last text."""
    S, F, n, t = c["S"], c["frame"], c["texts"], c["text"]
    nf = max(0, (S - n * t) // F)
    m, left = [], nf
    for i in range(n):
        f = left // (n - i)
        left -= f
        m += [np.zeros(t + (S - n * t - nf * F if i == n - 1 else 0), np.uint8), np.ones(f * F, np.uint8)]
    return np.concatenate(m)[:S]


def heads(c):
    """Per-head patterns as an offline search leaves them, in turn over the heads."""
    F = c["frame"]
    qb = C.qboundary_head({0: C.ashape(128, 1024), 1: C.vslash(1000, 1024)})
    b2d = C.boundary2d_head({0: C.ashape(128, 1024), 1: C.grid_frame(F)}, {(0, 1): C.vert(256), (1, 0): C.vert(256)})
    grid, vs = C.global_head(C.grid_window(F)), C.global_head(C.vslash(1000, 1024))
    kinds = {
        "grid": [C.global_head(C.grid_frame(F))],
        "mixed": [grid, C.global_head(C.ashape(128, 1024)), vs],
        "modal": [qb, b2d, grid, vs],
        "sinks": [grid, C.global_head(C.ashape(128, 8192)), C.global_head(C.vslash(200, 64))],
        "long": [grid, C.global_head(C.ashape(128, 4096)), vs, qb, b2d],
        "qbgrid": [C.qboundary_head({0: C.ashape(128, 4096), 1: C.grid_window(F)})],
    }[c["family"]]
    return [kinds[h % len(kinds)] for h in range(c["Hq"])]


_ctx = None


def context():
    """The one handle that a program keeps."""
    global _ctx
    if _ctx is None:
        _ctx = mmi.Ctx(0)
    return _ctx


def qkv(c, seed, mod, family):
    """Seeded Q/K/V with the structure of video prompts (periodic frames, line
    slots, locally correlated text, sinks)."""
    rng = np.random.default_rng(seed)
    sig = [c["frame"]] * c["Hkv"]
    if family in ("mixed", "qbgrid"):              # the searched strides differ from the frame size by a few tokens
        sig = [max(2, c["frame"] + int(rng.integers(-4, 5))) for _ in sig]
    st = generate.Structure(sigma=sig, amp=1.5 if family == "sinks" else 2.0, v_embed=family in ("grid", "mixed"),
                            text_amp=1.0 if family in ("modal", "search") else 0.0,
                            sink_frac=0.01 if family == "sinks" else 0.0)
    st.line_slot = [int(rng.integers(0, s)) for s in sig]
    wl = generate.Workload("case", c["S"], c["Hq"], c["Hkv"], mod, [], st, int(seed), frame=c["frame"])
    return generate.make_qkv(wl, DEV)


def fused(q, k, v):
    """The same values as views of one [S, (Hq + 2 Hkv) 128] projection output."""
    S, Hq, Hkv = q.shape[0], q.shape[1], k.shape[1]
    x = torch.cat([q.reshape(S, -1), k.reshape(S, -1), v.reshape(S, -1)], 1).contiguous().view(S, Hq + 2 * Hkv, D)
    return x[:, :Hq], x[:, Hq:Hq + Hkv], x[:, Hq + Hkv:]


def grid_order(L, s, p):
    """Coordinates [0, L) grouped by phase c mod s, phases p+1, ..., p."""
    c = torch.arange(L, device=DEV)
    return torch.argsort(((c - p - 1) % s) * (L // s + 2) + c // s, stable=True)


def prepare(c, seed):
    s = {"c": c}
    if c["what"] == "permute":
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        draw_ = lambda h: torch.randn(c["S"], h, D, device=DEV, generator=g).to(torch.bfloat16)  # noqa: E731
        s["q"], s["k"], s["v"] = draw_(c["Hq"]), draw_(c["Hkv"]), draw_(c["Hkv"])
        rng = np.random.default_rng(seed)
        s["perm"] = [grid_order(c["S"], c["frame"], int(rng.integers(0, c["frame"]))).int() for _ in range(c["Hkv"])]
        s["qs"], s["ks"], s["vs"] = (torch.empty(t.shape[1], c["S"], D, device=DEV, dtype=torch.bfloat16)
                                     for t in (s["q"], s["k"], s["v"]))
        s["o"] = torch.empty_like(s["q"])
        return s
    if c["what"] in ("natten", "dense"):
        S = c["T"] * c["H"] * c["W"] if c["what"] == "natten" else c["S"]
        Hkv = c["Hq"] if c["what"] == "natten" else c["Hkv"]
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        s["q"], s["k"], s["v"] = (torch.randn(S, h, D, device=DEV, generator=g).to(torch.bfloat16)
                                  for h in (c["Hq"], Hkv, Hkv))
        s["prob"] = mmi.Problem(S, c["Hq"], Hkv, None)
        if c["what"] == "natten":
            op = C.natten((c["T"], c["H"], c["W"]), (c["wt"], c["wh"], c["ww"]), (c["tt"], c["th"], c["tw"]))
            s["heads"] = [C.global_head(op)] * c["Hq"]
    else:
        mod = layout(c)
        s["mod"] = mod
        q, k, v = qkv(c, seed, mod, c.get("family", "search"))
        strides = None
        if c.get("fused"):
            q, k, v = fused(q, k, v)
            strides = {n: (t.stride(0), t.stride(1)) for n, t in (("q", q), ("k", k), ("v", v))}
            strides["o"] = (c["Hq"] * D, D)
        s["q"], s["k"], s["v"] = q, k, v
        s["prob"] = mmi.Problem(c["S"], c["Hq"], c["Hkv"], mod, strides)
        if c["what"] == "search":
            s["cands"] = [op for _, op in search_space.intra_candidates(c["frame"])]
            s["xc"] = [op for _, op in search_space.cross_candidates()]
            s["target"] = search_space.budget_op()
        else:
            s["heads"] = heads(c)
    if DEV == "cuda":
        s["ctx"] = context()
    S = s["q"].shape[0]
    s["o"] = torch.empty(S, c["Hq"], D, device=DEV, dtype=torch.bfloat16)
    s["lse"] = torch.empty(c["Hq"], S, device=DEV, dtype=torch.float32) if c.get("lse") else None
    return s


def run(s):
    c, what = s["c"], s["c"]["what"]
    q, k, v, o, lse = s["q"], s["k"], s["v"], s["o"], s.get("lse")
    if what == "permute":
        G = c["Hq"] // c["Hkv"]
        for h in range(c["Hkv"]):
            mmi.mmi_permute_rows(k[:, h], s["ks"][h], s["perm"][h])
            mmi.mmi_permute_rows(v[:, h], s["vs"][h], s["perm"][h])
        for h in range(c["Hq"]):
            mmi.mmi_permute_rows(q[:, h], s["qs"][h], s["perm"][h // G])
            mmi.mmi_unpermute_rows(s["qs"][h], o[:, h], s["perm"][h // G])
        return [s["qs"], s["ks"], s["vs"], o]
    if what == "search":
        _, r = mmi.mmi_search(s["ctx"], s["prob"], q, k, v, s["cands"], s["xc"], s["target"])
        # the cross step's and the last step's figures are those of whichever candidates the first step chose, where
        # near-equal errors may fall either way; the candidates' own figures and budgets depend on the inputs alone
        return {n: r[n] for n in ("budget1", "step1_cost", "step1_err", "budget3", "step3g_cost", "step3g_err")}
    if what == "dense":
        mmi.mmi_dense_attention(s["ctx"], s["prob"], q, k, v, o, lse)
    elif c.get("entry") == "call":
        mmi.mmi_attention(s["ctx"], s["prob"], s["heads"], q, k, v, o, lse)
    elif c.get("entry") == "noalloc":
        mmi.mmi_attention_noalloc(s["ctx"], s["prob"], s["heads"], q, k, v, o, lse)
    else:
        plan = mmi.Plan(s["ctx"], s["prob"], s["heads"], q, k)
        plan.execute(q, k, v, o, lse)
        plan.destroy()
    return [o] if lse is None else [o, lse]


# ------------------------------------------------------------------ work and tolerance
def pairs(op, n):
    """Query-key pairs that an op needs over n causal queries and keys, to the
    block where that is known without the data (a Vertical-Slash query block
    is taken to need a key block per slash and one per eight verticals: at
    256K and 1M tokens the selected blocks come to within a quarter of that)."""
    full = n * (n + 1) / 2
    if op.kind == C.OP_ASHAPE:
        w = min(n, op.sink + op.local + B)
        return w * (w + 1) / 2 + (n - w) * w
    if op.kind == C.OP_GRID:                       # same phase, the line phase's columns and rows, the own block
        s = op.stride_lo
        return min(full, full * 3 / s + n * B)
    if op.kind == C.OP_VSLASH:
        w = min(n, B * (op.n_slash + op.n_vertical / 8))
        return w * (w + 1) / 2 + (n - w) * w
    return full


def layer_pairs(h, mod):
    nt, nv = int((mod == 0).sum()), int((mod == 1).sum())
    n = nt + nv
    if h.kind == C.HEAD_GLOBAL:
        return pairs(h.op, n)
    p0, p1 = pairs(h.intra_op(0), nt), pairs(h.intra_op(1), nv)
    if h.kind == C.HEAD_QBOUNDARY:
        f0, f1 = nt / max(n, 1), nv / max(n, 1)
        return pairs(h.intra_op(0), n) * f0 + pairs(h.intra_op(1), n) * f1
    return p0 + p1 + min(nt * nv / 2, (nt + nv) * 256)


def work(c):
    what = c["what"]
    S = c["T"] * c["H"] * c["W"] if what == "natten" else c["S"]
    Hkv = c["Hq"] if what == "natten" else c["Hkv"]
    row = 2 * D
    if what == "permute":
        # K, V, Q gathered once and the gathered Q rows scattered; the maps once each
        return {"bytes": 2 * S * row * (2 * Hkv + 2 * c["Hq"]) + 4 * S * Hkv, "flops": 0}
    io = S * row * (2 * c["Hq"] + 2 * Hkv) + (4 * S * c["Hq"] if c.get("lse") else 0)
    if what == "natten":
        n = S * c["wt"] * c["wh"] * c["ww"] * c["Hq"]
    elif what == "dense":
        n = S * (S + 1) / 2 * c["Hq"]
    elif what == "search":
        # every candidate inside the modalities and over all rows, six cross candidates, two dense references
        mod = layout(c)
        nt, nv = int((mod == 0).sum()), int((mod == 1).sum())
        ops = [op for _, op in search_space.intra_candidates(c["frame"])]
        n = sum(pairs(o, nt) + pairs(o, nv) + pairs(o, S) for o in ops) + 8 * S * (S + 1) / 2
        n *= c["Hq"]
        io = S * row * (c["Hq"] + 2 * Hkv)
    else:
        mod = layout(c)
        n = sum(layer_pairs(h, mod) for h in heads(c))
    return {"bytes": io, "flops": 4 * D * n}


def tolerance(c):
    if c["what"] == "permute":
        return "exact"
    if c["what"] == "search":
        return {"rel": 1e-3, "max": 0.1, "differ": 0.005}
    # bf16 outputs off by 1.3e-3 to 2.3e-3 of exact(); a tied column or diagonal may move a block's rows by more
    return {"rel": 8e-3, "max": 0.5}


# ------------------------------------------------------------------ 64-bit reference
SCALE = 1.0 / math.sqrt(D)


def pad(order):
    n = -len(order) % B
    return torch.cat([order, torch.full((n,), -1, device=DEV, dtype=order.dtype)]) if n else order


def estimate(q, k, rows):
    """softmax over the causal keys of the given rows: [rows, S] in float64."""
    S = k.shape[0]
    a = q[rows].double() @ k.double().t() * SCALE
    a.masked_fill_(torch.arange(S, device=DEV)[None] > rows[:, None], -math.inf)
    return torch.softmax(a, 1)


def topk(x, n):
    n = min(n, len(x))
    m = torch.zeros(len(x), dtype=torch.bool, device=DEV)
    m[torch.sort(x.float(), descending=True, stable=True).indices[:n]] = True
    return m


def diagonals(a, coord, L):
    u = torch.zeros(L, dtype=torch.float64, device=DEV)
    for r in range(len(coord)):
        x = int(coord[r])
        u[:x + 1] += a[r, :x + 1].flip(0)
    return u


def stride_phase(v, op):
    """(stride, phase) of the largest mean fold; a later stride must win by 2%."""
    L, best, got = len(v), np.float32(0), None
    v = v.float()
    for s in range(max(1, op.stride_lo), min(op.stride_hi, L // 2) + 1):
        idx = torch.arange(L, device=DEV) % s
        f = torch.zeros(s, dtype=torch.float64, device=DEV).index_add_(0, idx, v.double())
        f = (f / torch.bincount(idx, minlength=s)).float()
        p = int(f.argmax())
        x = np.float32(f[p].item())
        if x > best * np.float32(1.02):
            best, got = x, (s, p)
    return got


def predicate(op, a, coord, L):
    """pred(q, k) on coordinates, and the key order of a Grid op; `a`: the
    estimate over the op's first len(a[0]) key coordinates, its rows' coordinates `coord`."""
    if op.kind == C.OP_ASHAPE:
        return (lambda q, k: (k < op.sink) | (q - k < op.local)), None
    if op.kind == C.OP_VSLASH:
        V = torch.zeros(L, dtype=torch.bool, device=DEV)
        U = torch.zeros(L, dtype=torch.bool, device=DEV)
        V[:a.shape[1]] = topk(a.sum(0), op.n_vertical)
        U[:a.shape[1]] = topk(diagonals(a, coord, a.shape[1]), op.n_slash)
        return (lambda q, k: V[k] | U[(q - k).clamp_(min=0)]), None
    if op.kind == C.OP_GRID:
        got = stride_phase(a.sum(0), op)
        if got:
            s, p = got
            h, v, d = op.use_h, op.use_v, op.use_s
            return (lambda q, k: ((q % s == k % s) & d) | ((k % s == p) & v) | ((q % s == p) & h)), got
    return (lambda q, k: (k >= 0) | (q >= 0)), None


def lift(qpos, kpos, qc, kc, pred, own):
    """[query blocks, key blocks]: some pair with k <= q satisfies pred, or the key block holds a row's own key."""
    nq, nk = len(qpos) // B, len(kpos) // B
    sel = torch.zeros(nq, nk, dtype=torch.bool, device=DEV)
    step = max(1, (1 << 27) // max(1, len(kpos)) // B)
    for i in range(0, nq, step):
        r = slice(i * B, min(nq, i + step) * B)
        m = pred(qc[r, None], kc[None]) & (kpos[None] <= qpos[r, None]) & (kpos >= 0)[None] & (qpos[r] >= 0)[:, None]
        sel[i:i + step] = m.view(-1, B, nk, B).any(3).any(1)
    if own:
        S = int(max(qpos.max(), kpos.max())) + 1
        slot = torch.full((S,), -1, dtype=torch.long, device=DEV)
        live = kpos >= 0
        slot[kpos[live]] = torch.nonzero(live)[:, 0]
        for x in range(B):
            p = qpos[x::B]
            ok = p >= 0
            t = slot[p.clamp(min=0)]
            ok &= t >= 0
            sel[torch.nonzero(ok)[:, 0], t[ok] // B] = True
    return sel


def attend(qpos, kpos, sel, q, k, v, o, lse, causal=True):
    """Masked softmax of the rows qpos over the selected key blocks, written to o / lse at the rows."""
    nq = len(qpos) // B
    step = 16
    for i in range(0, nq, step):
        sl = sel[i:i + step]
        cols = torch.nonzero(sl.any(0))[:, 0]
        ks = (cols[:, None] * B + torch.arange(B, device=DEV)).reshape(-1)
        kp = kpos[ks]
        ks, kp = ks[kp >= 0], kp[kp >= 0]
        r = torch.arange(i * B, min(nq, i + step) * B, device=DEV)
        qp = qpos[r]
        r, qp = r[qp >= 0], qp[qp >= 0]
        if not len(r):
            continue
        a = q[qp].double() @ k[kp].double().t()
        a *= SCALE
        m = sl[r // B - i][:, ks // B]
        if causal:
            m &= kp[None] <= qp[:, None]
        a.masked_fill_(~m, -math.inf)
        l = torch.logsumexp(a, 1)
        o[qp] = torch.exp_(a.sub_(l[:, None])) @ v[kp].double()
        if lse is not None:
            lse[qp] = l


def ident(n):
    return torch.arange(n, device=DEV)


def final_rows(mod, m):
    """The last <= 64 positions of the last run of modality m."""
    p = np.nonzero(mod == m)[0]
    cut = np.nonzero(np.diff(p) != 1)[0]
    run_ = p[cut[-1] + 1:] if len(cut) else p
    return torch.as_tensor(run_[-64:].copy(), device=DEV)


def exact_head(h, mod, q, k, v, o, lse):
    S = k.shape[0]
    if h.kind == C.HEAD_GLOBAL:
        rows = ident(S)[-64:]
        a = estimate(q, k, rows) if h.op.kind in (C.OP_GRID, C.OP_VSLASH) else None
        pred, grid = predicate(h.op, a, rows, S)
        pos = pad(grid_order(S, *grid) if grid else ident(S))
        sel = lift(pos, pos, pos.clamp(min=0), pos.clamp(min=0), pred, True)
        return attend(pos, pos, sel, q, k, v, o, lse)
    mods = [m for m in range(C.MAX_MODALITIES) if (mod == m).any()]
    where = {m: torch.as_tensor(np.nonzero(mod == m)[0], device=DEV) for m in mods}
    if h.kind == C.HEAD_QBOUNDARY:
        for m in mods:
            op, rows = h.intra_op(m), final_rows(mod, m)
            a = None
            if op.kind in (C.OP_GRID, C.OP_VSLASH):
                a = estimate(q, k, rows)[:, :int(rows[-1]) + 1]
            pred, grid = predicate(op, a, rows, S)
            order = grid_order(S, *grid) if grid else ident(S)
            kpos = pad(order)
            mine = torch.as_tensor(mod == m, device=DEV)
            qpos = pad(order[mine[order]])
            sel = lift(qpos, kpos, qpos.clamp(min=0), kpos.clamp(min=0), pred, True)
            attend(qpos, kpos, sel, q, k, v, o, lse)
        return None
    local = torch.zeros(S, dtype=torch.long, device=DEV)
    intra, order = {}, {}
    for m in mods:
        local[where[m]] = ident(len(where[m]))
        op, rows, a = h.intra_op(m), final_rows(mod, m), None
        if op.kind in (C.OP_GRID, C.OP_VSLASH):
            a = estimate(q, k, rows)[:, where[m]]
        intra[m], grid = predicate(op, a, local[rows], len(where[m]))
        order[m] = pad(where[m][grid_order(len(where[m]), *grid)] if grid else where[m])
    for m in mods:
        sel, keys = [], torch.cat([order[x] for x in mods])
        for x in mods:
            pred, op = intra[m], h.cross_op(m, x)
            if x != m and op.kind == C.OP_VERT:
                rows = final_rows(mod, m)
                n = int((where[x] <= rows[-1]).sum())
                V = torch.zeros(len(where[x]), dtype=torch.bool, device=DEV)
                if n:
                    V[:n] = topk(estimate(q, k, rows)[:, where[x][:n]].sum(0), op.n_vertical)
                pred = lambda qq, kk, V=V: V[kk] | (qq < 0)  # noqa: E731
            elif x != m:
                pred = lambda qq, kk, on=op.kind == C.OP_DENSE: (kk >= 0) & (qq >= 0) & on  # noqa: E731
            sel.append(lift(order[m], order[x], local[order[m].clamp(min=0)], local[order[x].clamp(min=0)], pred, x == m))
        attend(order[m], keys, torch.cat(sel, 1), q, k, v, o, lse)
    return None


def exact_natten(c, q, k, v, o):
    n, w, t = (c["T"], c["H"], c["W"]), (c["wt"], c["wh"], c["ww"]), (c["tt"], c["th"], c["tw"])
    nt = [-(-a // b) for a, b in zip(n, t)]
    # position of every (tile, token of the tile), -1 past the border
    grids = torch.meshgrid(*[torch.arange(x, device=DEV) for x in (*nt, *t)], indexing="ij")
    co = [grids[a] * t[a] + grids[3 + a] for a in range(3)]
    pos = (co[0] * n[1] + co[1]) * n[2] + co[2]
    bad = (co[0] >= n[0]) | (co[1] >= n[1]) | (co[2] >= n[2])
    pos = torch.where(bad, torch.full_like(pos, -1), pos).reshape(-1)
    sel = torch.ones(1, 1, dtype=torch.bool, device=DEV)
    for a in range(3):                               # per axis: key tiles that meet the union of a query tile's windows
        s = torch.zeros(nt[a], nt[a], dtype=torch.bool, device=DEV)
        for x in range(n[a]):
            lo = min(max(x - w[a] // 2, 0), n[a] - w[a])
            s[x // t[a], lo // t[a]:(lo + w[a] - 1) // t[a] + 1] = True
        sel = (sel[:, None, :, None] & s[None, :, None, :]).reshape(sel.shape[0] * nt[a], -1)
    attend(pos, pos, sel, q, k, v, o, None, causal=False)


def exact(c, seed):
    what = c["what"]
    if what == "search" or (what == "layer" and c["S"] > 140000):
        return None                                  # tens of seconds and more in 64 bits
    s = prepare(c, seed)
    q, k, v = s["q"], s["k"], s["v"]
    if what == "permute":
        G = c["Hq"] // c["Hkv"]
        p = [x.long() for x in s["perm"]]
        return [torch.stack([q[:, h][p[h // G]] for h in range(c["Hq"])]),
                torch.stack([k[:, h][p[h]] for h in range(c["Hkv"])]),
                torch.stack([v[:, h][p[h]] for h in range(c["Hkv"])]), q]
    S, Hq = q.shape[0], c["Hq"]
    G = Hq // k.shape[1]
    O = torch.zeros(S, Hq, D, dtype=torch.float64, device=DEV)
    L = torch.zeros(Hq, S, dtype=torch.float64, device=DEV) if c.get("lse") else None
    for h in range(Hq):
        g = h // G
        args = q[:, h], k[:, g], v[:, g], O[:, h]
        if what == "natten":
            exact_natten(c, *args)
        elif what == "dense":
            nb = -(-S // B)
            sel = torch.ones(nb, nb, dtype=torch.bool, device=DEV).tril_()
            attend(pad(ident(S)), pad(ident(S)), sel, *args, None if L is None else L[h])
        else:
            exact_head(s["heads"][h], s["mod"], *args, None if L is None else L[h])
    return [O] if L is None else [O, L]
