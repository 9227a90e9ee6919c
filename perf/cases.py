"""Performance cases: the stage calls that a serving program makes, over the sizes it makes them at.

The program behind these cases serves a looped language model with continuous depth batching: prompts enter
through chunked prefill, every decode token runs loop steps over a mixed-depth batch until it exits, and exits go
through the coda (and the next token through the prelude).  Widths are those of the two model families that the
tests and the benchmark use (Ouro 1.4B: d 2048, 16 x 128 heads, 24 core layers, r_max 4; Huginn 3.5B: d 5280,
55 x 96 heads, 2-4-2 layers with the injection adapter, r_max 32).  Most cases take a few layers of a model, which
is what one layer of the whole costs times that many; one takes the whole 24-layer loop step.

A case is a dict:
  call      "step" (cdb_loop_step / cdb_loop_step_gated), "prefill", "coda" or "prelude"
  model     "ouro" or "huginn"
  layers    core layers kept (the whole core: 24, 4)
  rows      rows of the call (prefill: tokens of the chunk)
  lo, hi    step, coda, prelude: positions are drawn from [lo, hi]; prefill: the chunk starts at position lo
  gate      step: exits decided on the device with the lookahead gate instead of replayed depths
  live      step: rows counted in device memory (0: the host's count), as a captured graph replays them
  loops     prefill: loop iterations (r_max) of the model
  logits    prefill: all rows' logits (else the last row's greedy id, as the serving driver asks for)
"""
from __future__ import annotations

import ctypes as C
import math

import numpy as np
import torch

import cdbgen
import paper_2608_09444_amd as cdb

MODELS = {"ouro": cdbgen.OURO, "huginn": cdbgen.HUGINN}
DEPTHS = {"ouro": cdbgen.OURO_DEPTHS, "huginn": cdbgen.WORKLOADS[3].depth}
NAMES = ("q", "k", "v", "o", "gate", "up", "down")


def _step(model, layers, rows, lo, hi, gate=False, live=0):
    return {"call": "step", "model": model, "layers": layers, "rows": rows, "lo": lo, "hi": hi, "gate": gate,
            "live": live}


def _prefill(model, layers, rows, lo, loops, logits):
    return {"call": "prefill", "model": model, "layers": layers, "rows": rows, "lo": lo, "loops": loops,
            "logits": logits}


def _boundary(call, rows, lo, hi):
    return {"call": call, "model": "huginn", "layers": 1, "rows": rows, "lo": lo, "hi": hi}


def listed():
    return [
        # one user's token: the smallest call a server makes
        dict(_step("ouro", 4, 1, 100, 800), name="step_ouro_1"),
        # a handful of long-context requests
        dict(_step("ouro", 4, 6, 2048, 4223), name="step_ouro_6_long"),
        # the partly filled batch at the end of a decode, exits decided by the gate
        dict(_step("ouro", 4, 23, 16, 800, gate=True), name="step_ouro_23_gated"),
        # the benchmark's batch: 64 rows in the decode range of a 512-token prompt, the whole core
        dict(_step("ouro", 24, 64, 512, 767), name="step_ouro_64_whole"),
        # a step of capacity 128 with 100 rows in it, counted on the device as a graph replay does
        dict(_step("ouro", 4, 128, 100, 767, live=100), name="step_ouro_100_of_128"),
        # the largest decode batch of the long-context workload
        dict(_step("ouro", 2, 256, 2048, 4223), name="step_ouro_256_long"),
        # the Huginn-shaped refill batch: the whole core with its adapter, shared K/V
        dict(_step("huginn", 4, 128, 256, 767), name="step_huginn_128"),
        # the same model with few requests
        dict(_step("huginn", 4, 9, 256, 767), name="step_huginn_9"),
        # a full prompt chunk as the serving driver runs it
        dict(_prefill("ouro", 4, 512, 0, 4, False), name="prefill_ouro_512"),
        # the ragged last chunk of a long prompt, with every row's logits (scoring)
        dict(_prefill("ouro", 4, 333, 1500, 4, True), name="prefill_ouro_333_later"),
        # a Huginn-shaped prompt through prelude, two core loops and coda
        dict(_prefill("huginn", 4, 300, 0, 2, True), name="prefill_huginn_300"),
        # the boundary batch of exiting tokens: two layers, the 65536-row LM head, greedy ids
        dict(_boundary("coda", 32, 256, 767), name="coda_huginn_32"),
    ]


def draw(rng):
    """Sizes log-uniform over the ranges of the listed cases."""
    def logint(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(("step", "step", "step", "step", "prefill", "prefill", "boundary"))
    if kind == "step":
        model = rng.choice(("ouro", "ouro", "huginn"))
        rows = logint(1, 256 if model == "ouro" else 128)
        lo = logint(16, 2048 if model == "ouro" else 512)
        hi = min(4223, 2 * lo + rng.randrange(256))
        layers = 2 if rows * hi > 200_000 else rng.choice((2, 3, 4))
        return _step(model, layers, rows, lo, hi, gate=rng.random() < 0.3,
                     live=max(1, rows - rng.randrange(1 + rows // 3)) if rng.random() < 0.3 else 0)
    if kind == "prefill":
        if rng.random() < 0.7:
            return _prefill("ouro", rng.choice((2, 3, 4)), logint(17, 512), rng.choice((0, logint(16, 3000))), 4,
                            rng.random() < 0.5)
        return _prefill("huginn", 4, logint(17, 300), rng.choice((0, logint(16, 700))), 2, rng.random() < 0.5)
    return _boundary(rng.choice(("coda", "coda", "prelude")), logint(1, 128), 16, logint(64, 767))


# ------------------------------------------------------------------ inputs

def _shape(case):
    s = MODELS[case["model"]]
    kw = {"n_core": case["layers"]}
    if case["call"] == "prefill":
        kw["r_max"] = case["loops"]
    elif case["call"] == "prelude":
        kw["n_coda"] = 0
    elif case["call"] == "coda":
        kw["n_prelude"] = 0
    return cdbgen.shrink(s, **kw)


def _weights(s, seed):
    """Plain bf16 weights N(0, 0.02) on the device: {tensor: [out][in]} with one dict per layer."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000 + 1)

    def w(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)

    top = {"embed": w(s.vocab, s.d), "lm_head": w(s.vocab, s.d), "w_exit": w(s.d),
           "adapter": w(s.d, 2 * s.d) if s.injection else None}
    top["layers"] = [{n: w(*shp) for n, shp in cdbgen.layer_shapes(s).items()} for _ in range(s.n_layers)]
    return top


def _pack(s, w):
    desc = cdb.make_desc(s)
    packed = torch.empty(cdb.cdb_packed_weight_bytes(desc), dtype=torch.uint8, device="cuda")
    ptrs = [lw[n].data_ptr() for lw in w["layers"] for n in NAMES]
    arr = (C.c_void_p * max(1, len(ptrs)))(*ptrs)
    plain = cdb.cdb_plain_weights(w["embed"].data_ptr(), w["lm_head"].data_ptr(), w["w_exit"].data_ptr(),
                                  w["adapter"].data_ptr() if s.injection else None,
                                  C.cast(arr, C.POINTER(C.c_void_p)))
    cdb.cdb_pack_weights(desc, plain, packed)
    torch.cuda.synchronize()  # the plain weights are dropped after this
    return desc, packed


def _rows(case, s, seed):
    """The call's rows: one per sequence, mid-decode, loop indices below their size-biased depths."""
    return cdbgen.decode_snapshot(case["rows"], DEPTHS[case["model"]], s.r_max, case["lo"], case["hi"],
                                  seed=seed * 7 + 2)


def _page_table(case, s, rows):
    """(page table, pages per pool).  Ouro-shaped steps: the depth-indexed cache, each row's own loop plane over its
    context and the page at its position of every deeper plane (where copy-on-exit writes).  Huginn-shaped steps: the
    shared layout, all loop planes on one page.  Prefill: every plane of one sequence."""
    R = s.r_max
    if case["call"] == "prefill":
        n = cdbgen.pages_for(case["lo"] + case["rows"])
        pt = np.full((1, R + 2, n), -1, np.int32)
        if s.n_prelude:
            pt[0, 0] = np.arange(n)
        pt[0, 1:R + 1] = np.arange(n * R).reshape(n, R).T
        if s.n_coda:
            pt[0, R + 1] = np.arange(n)
        return pt, (n, n * R, n)
    pos, c = rows["pos"], rows["c"]
    n_seq, max_pages = len(pos), case["hi"] // 16 + 1
    pt = np.full((n_seq, R + 2, max_pages), -1, np.int32)
    nxt = 0
    for i in range(n_seq):
        n = int(pos[i]) // 16 + 1
        if case["call"] != "step":
            pt[i, 0 if case["call"] == "prelude" else R + 1, :n] = np.arange(nxt, nxt + n)
        elif case["model"] == "huginn":
            pt[i, 1:R + 1, :n] = np.arange(nxt, nxt + n)
        else:
            pt[i, c[i] + 1, :n] = np.arange(nxt, nxt + n)
            deeper = R - 1 - int(c[i])
            pt[i, c[i] + 2:R + 1, n - 1] = np.arange(nxt + n, nxt + n + deeper)
            nxt += deeper
        nxt += n
    pages = n_seq * (max_pages + R - 1)  # what the longest rows of these ranges need
    return pt, {"step": (0, pages, 0), "prelude": (pages, 0, 0), "coda": (0, 0, pages)}[case["call"]]


def _cache(s, pt, pages, seed):
    kv = cdb.PagedKV(s, pt.shape[0], pt.shape[2], *pages, fill="random")
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000 + 2)
    for pool in (kv.pre, kv.core, kv.coda):
        pool.normal_(0.0, 1.0, generator=g)
    kv.page_table.copy_(torch.from_numpy(pt))
    return kv


def _state(s, n, seed):
    st = cdb.State(s, n)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000 + 3)
    st.h.normal_(0.0, 1.0, generator=g)
    if st.e is not None:
        st.e.normal_(0.0, 1.0, generator=g)
    return st


def _tokens(case, s, seed):
    return torch.from_numpy(cdbgen.prompt_ids(s.vocab, 1, case["rows"], seed=seed * 7 + 3)[0]).cuda()


THRESHOLD = {0: 0.9, 1: 1.0}  # exit scores: sigmoid above, convergence distance below


def prepare(case, seed):
    s = _shape(case)
    w = _weights(s, seed)
    desc, packed = _pack(s, w)
    del w
    n = case["rows"]
    rows_np = None if case["call"] == "prefill" else _rows(case, s, seed)
    pt, pages = _page_table(case, s, rows_np)
    kv = _cache(s, pt, pages, seed)
    st = {"case": case, "shape": s, "model": cdb.cdb_model(packed.data_ptr(), desc), "packed": packed, "kv": kv,
          "ws": cdb.Workspace(desc, n)}
    if case["call"] == "prefill":
        st["tokens"] = _tokens(case, s, seed)
        st["logits"] = torch.empty((n, s.vocab), dtype=torch.float32, device="cuda") if case["logits"] else None
        st["ids"] = torch.empty(n if case["logits"] else 1, dtype=torch.int32, device="cuda")
        return st
    st["state"] = _state(s, n, seed)
    live = None
    if case.get("live"):
        live = torch.tensor([case["live"]], dtype=torch.int32, device="cuda")
    st["rows"] = cdb.Rows(rows_np["slot"], rows_np["seq"], rows_np["pos"], rows_np["c"], rows_np["depth"],
                          d_n_rows=live)
    if case["call"] == "step":
        st["out"] = cdb.StepOut(n)
        st["gate"] = cdb.Gate(THRESHOLD[s.exit_kind], True, n) if case["gate"] else None
    elif case["call"] == "coda":
        st["logits"] = torch.empty((n, s.vocab), dtype=torch.float32, device="cuda")
        st["ids"] = torch.empty(n, dtype=torch.int32, device="cuda")
    else:
        st["tokens"] = _tokens(case, s, seed)
    return st


# pools up to this many elements are returned whole (a decode step writes one entry per row into them)
POOL_RETURNED = 1 << 29


def _pool(case, kv):
    p = {"step": kv.core, "prefill": kv.core, "coda": kv.coda, "prelude": kv.pre}[case["call"]]
    return p if p.numel() <= POOL_RETURNED else None


def run(state):
    """Greedy ids are not among the outputs: on random weights a rounding decides some of them; they follow from the
    logits, which are."""
    case, kv, ws = state["case"], state["kv"], state["ws"].buf
    if case["call"] == "prefill":
        cdb.cdb_prefill(state["model"], kv.c, 0, case["lo"], state["tokens"], state["logits"], state["ids"], ws)
        return {"logits": state["logits"], "pool": _pool(case, kv)}
    st, rows = state["state"], state["rows"]
    if case["call"] == "coda":
        cdb.cdb_boundary_coda(state["model"], kv.c, st.c, rows.c, state["logits"], state["ids"], ws)
        return {"logits": state["logits"], "pool": _pool(case, kv)}
    if case["call"] == "prelude":
        cdb.cdb_boundary_prelude(state["model"], kv.c, st.c, rows.c, state["tokens"], ws)
        return {"h": st.h, "e": st.e, "pool": _pool(case, kv)}
    out = state["out"]
    if state["gate"] is not None:
        cdb.cdb_loop_step_gated(state["model"], kv.c, st.c, rows.c, state["gate"].c, out.c, ws)
    else:
        cdb.cdb_loop_step(state["model"], kv.c, st.c, rows.c, out.c, ws)
    return {"h": st.h, "score": out.score, "mask": out.mask, "cont": out.cont, "exited": out.exited,
            "counts": out.counts, "exit_next": out.exit_next, "pool": _pool(case, kv)}


# ------------------------------------------------------------------ what a pass cannot do without

def _layer_params(s):
    return 4 * s.d * s.d + 3 * s.d * s.d_ff


def work(case):
    s = _shape(case)
    P, d, R = _layer_params(s), s.d, s.r_max
    kv_tok = 2 * d * 2  # K and V of one position in one layer
    if case["call"] == "prefill":
        n, p0 = case["rows"], case["lo"]
        passes = s.n_prelude + R * s.n_core + s.n_coda
        heads = n if case["logits"] else 1
        adapter = 2 * d * d * s.injection
        flops = 2 * n * (P * passes + adapter * R) + 4 * d * passes * (n * p0 + n * (n + 1) // 2) + 2 * heads * s.vocab * d
        weights = s.n_layers * P + adapter + s.vocab * d
        return {"bytes": 2 * weights + passes * kv_tok * (p0 + n) + n * d * 2 + (n * s.vocab * 4 if case["logits"] else 4),
                "flops": flops}
    rows = _rows(case, s, 1)  # the same distribution at every seed
    n = case.get("live") or case["rows"]
    ctx = int((rows["pos"][:n].astype(np.int64) + 1).sum())
    if case["call"] == "step":
        layers, extra = s.n_core, 2 * d * d * s.injection + d
        ex = (rows["c"][:n] + 1 == rows["depth"][:n]) & (not case["gate"]) & (case["model"] == "ouro")
        other = int(((R - rows["depth"][:n]) * ex).sum()) * 2 * kv_tok * layers + n * d * 4 * (2 + s.injection)
    elif case["call"] == "coda":
        layers, extra, other = s.n_coda, s.vocab * d, n * d * 4 + n * s.vocab * 4
    else:
        layers, extra, other = s.n_prelude, 0, n * d * (2 + 4 * 2)
    return {"bytes": 2 * (layers * P + extra) + layers * kv_tok * (ctx + n) + other,
            "flops": 2 * n * (layers * P + extra) + 4 * d * layers * ctx}


def tolerance(case):
    """Activations, K/V and the inputs of matrix products are bf16 between fp32 sums, so another summation order flips
    some of their roundings and every layer after sees that.  Measured against 64-bit arithmetic without those
    roundings: 3.3e-3 after 4 Ouro-shaped layers, 6.2e-3 after the Huginn-shaped core, 8.7e-3 after 24 layers, 1.0e-2 to
    1.5e-2 in prefills (up to 16 layer passes and the LM head)."""
    rel = 0.014 if case["call"] == "step" and case["model"] == "ouro" and case["layers"] <= 4 else 0.025
    if case["call"] == "prefill" or case["layers"] > 4:
        rel = 0.03
    return {"rel": rel, "max": 12 * rel, "differ": 0.01}


# ------------------------------------------------------------------ 64-bit reference

def _norm(x, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def _rope(x, pos, base):
    """x [rows][H][hd], rotate-half."""
    hd = x.shape[-1]
    inv = base ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=x.device) / hd)
    ang = pos.double()[:, None, None] * inv
    a, b = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _mm(x, w):
    return x @ w.double().t()


def _layer(s, lw, h, pos, attend):
    """One layer on h [rows][d]; attend(q, k, v) stores k and v and returns the attention output, all [rows][H][hd]."""
    n = h.shape[0]
    x = _norm(h, s.rms_eps)
    q, k, v = (_mm(x, lw[t]).view(n, s.n_heads, s.head_dim) for t in ("q", "k", "v"))
    o = attend(_rope(q, pos, s.rope_base), _rope(k, pos, s.rope_base), v)
    h = h + _mm(o.reshape(n, s.d), lw["o"])
    x = _norm(h, s.rms_eps)
    return h + _mm(torch.nn.functional.silu(_mm(x, lw["gate"])) * _mm(x, lw["up"]), lw["down"])


def _context(pool, layer, pids, n):
    """K and V [n][H][hd] in 64 bits of the first n positions on the given pages."""
    kv = pool[layer, pids].double()  # [pages][2][H][16][hd]
    kv = kv.permute(1, 0, 3, 2, 4).reshape(2, -1, kv.shape[2], kv.shape[4])
    return kv[0, :n], kv[1, :n]


def _decode_attend(s, pool, layer, pt, plane, pos, copies):
    def attend(q, k, v):
        out = torch.empty_like(q)
        for i in range(q.shape[0]):
            p = int(pos[i])
            pids = torch.as_tensor(pt[i, plane[i], :p // 16 + 1].astype(np.int64), device="cuda")
            K, V = _context(pool, layer, pids, p + 1)
            K[p], V[p] = k[i], v[i]
            sc = torch.softmax((K * q[i]).sum(-1) / math.sqrt(s.head_dim), 0)  # [n][H]
            out[i] = (V * sc[..., None]).sum(0)
        copies.append((layer, k, v))
        return out
    return attend


def _exact_rows(case, s, seed):
    w, rows = _weights(s, seed), _rows(case, s, seed)
    pt, pages = _page_table(case, s, rows)
    kv, st = _cache(s, pt, pages, seed), _state(s, case["rows"], seed)
    n = case.get("live") or case["rows"]
    pos = torch.from_numpy(rows["pos"][:n]).cuda()
    full, e = st.h.double(), None
    h_in = full[:n]
    written = []
    if case["call"] == "step":
        pool, plane = kv.core, rows["c"][:n] + 1
        h, layers = h_in, w["layers"][s.n_prelude:s.n_prelude + s.n_core]
        if s.injection:
            h = _mm(torch.cat([h, st.e.double()[:n]], 1), w["adapter"])
    elif case["call"] == "coda":
        pool, plane, h, layers = kv.coda, np.full(n, s.r_max + 1), h_in, w["layers"][s.n_prelude + s.n_core:]
    else:
        pool, plane, layers = kv.pre, np.zeros(n, np.int64), w["layers"][:s.n_prelude]
        h = w["embed"][_tokens(case, s, seed).long()].double()
    for l, lw in enumerate(layers):
        h = _layer(s, lw, h, pos, _decode_attend(s, pool, l, pt, plane, rows["pos"], written))
    if case["call"] == "prelude":
        e = h
    exp = None
    if pool.numel() <= POOL_RETURNED:
        exp = pool.double()
        for l, k, v in written:
            for i in range(n):
                p = int(rows["pos"][i])
                planes = [int(plane[i])]
                if case["call"] == "step" and not case["gate"] and rows["c"][i] + 1 == rows["depth"][i]:
                    planes = range(int(plane[i]), s.r_max + 1)
                for pl in planes:
                    exp[l, int(pt[i, pl, p // 16]), 0, :, p % 16] = k[i]
                    exp[l, int(pt[i, pl, p // 16]), 1, :, p % 16] = v[i]
    if case["call"] == "coda":
        return {"logits": _mm(_norm(h, s.rms_eps), w["lm_head"]), "pool": exp}
    if case["call"] == "prelude":
        return {"h": h, "e": e, "pool": exp}
    if s.exit_kind == 1:
        sc = (h - h_in).norm(dim=1)
    else:
        sc = torch.sigmoid(_norm(h, s.rms_eps) @ w["w_exit"].double())
    score = torch.zeros(case["rows"], dtype=torch.float64, device="cuda")
    score[:n] = sc
    full = full.clone()
    full[:n] = h
    # a gated step's exits write deeper planes' entries for rows that a rounding could decide
    return {"h": full, "score": score, "mask": None, "cont": None, "exited": None, "counts": None, "exit_next": None,
            "pool": None if case["gate"] else exp}


def _exact_prefill(case, s, seed):
    w = _weights(s, seed)
    pt, pages = _page_table(case, s, None)
    kv = _cache(s, pt, pages, seed)
    n, p0, R = case["rows"], case["lo"], s.r_max
    pos = torch.arange(p0, p0 + n, device="cuda")
    exp = kv.core.double() if kv.core.numel() <= POOL_RETURNED else None
    mask = torch.arange(p0 + n, device="cuda")[None, :] > pos[:, None]

    def attend_in(pool, layer, plane, to):
        def attend(q, k, v):
            pids = torch.as_tensor(pt[0, plane].astype(np.int64), device="cuda")
            K, V = _context(pool, layer, pids, p0 + n)
            K[p0:], V[p0:] = k, v
            if to is not None:
                pg = pids[(pos // 16)]
                to[layer, pg, 0, :, pos % 16] = k
                to[layer, pg, 1, :, pos % 16] = v
            out = torch.empty_like(q)
            for a in range(s.n_heads):
                sc = (q[:, a] @ K[:, a].t().contiguous()) / math.sqrt(s.head_dim)
                out[:, a] = torch.softmax(sc.masked_fill(mask, -math.inf), 1) @ V[:, a].contiguous()
            return out
        return attend

    h = w["embed"][_tokens(case, s, seed).long()].double()
    L0, L1 = s.n_prelude, s.n_prelude + s.n_core
    for l in range(L0):
        h = _layer(s, w["layers"][l], h, pos, attend_in(kv.pre, l, 0, None))
    e = h
    for r in range(1, R + 1):
        if s.injection:
            h = _mm(torch.cat([h, e], 1), w["adapter"])
        for l in range(s.n_core):
            h = _layer(s, w["layers"][L0 + l], h, pos, attend_in(kv.core, l, r, exp))
    for l in range(s.n_coda):
        h = _layer(s, w["layers"][L1 + l], h, pos, attend_in(kv.coda, l, R + 1, None))
    return {"logits": _mm(_norm(h, s.rms_eps), w["lm_head"]) if case["logits"] else None, "pool": exp}


def exact(case, seed):
    s = _shape(case)
    return _exact_prefill(case, s, seed) if case["call"] == "prefill" else _exact_rows(case, s, seed)
