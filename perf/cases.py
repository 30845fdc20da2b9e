"""The work that is timed when the speed of this library is compared between two builds.

Each case is one call (or the short chain of calls) that a program doing draft-guided
eviction makes, at Llama-3-8B KV geometry unless it says otherwise (32 query heads, 8 KV
heads, head dim 128, window 32, 2 draft rows, max-pool 7), or at the tiny fp32 geometry of
the c1 workload.  Kinds:

* ``step``    - the eviction of one layer, ``evict_layer`` with its defaults: score, select
                and compact, outputs and workspaces allocated by the call;
* ``score``   - scoring of a layer-major cache of one or many layers (``score``, or
                ``score_lse`` when the attention forward supplies the rows' log-sum-exp),
                with window + draft rows, draft rows only or window rows only;
* ``select``  - selection and compaction of every layer, each with its own budget
                (``select_compact_layers``), from given scores;
* ``h2o``     - H2O accumulated attention of one layer, row log-sum-exp computed or given;
* ``project`` - query capture, RoPE(x W^T), for the few scoring rows or a whole prompt;
* ``attend``  - the diagnostics on a compacted cache: ``cache_attention`` and, for rows
                inside the tail, ``evicted_mass``.

Inputs are standard normal queries, keys and values rounded to the storage type, with
16-key spans pulled toward the group's mean query where ``plant`` says so; scores handed to
the selection are means of log-normal draws, as a sum of softmax rows looks.
"""
import math

import torch

import paper_2609_33334_amd as dge

ROWS = {"window_draft": dge.ROWS_WINDOW_DRAFT, "draft": dge.ROWS_DRAFT, "window": dge.ROWS_WINDOW}
DEV = "cuda"


def listed():
    llama = dict(hq=32, hkv=8, d=128, dtype="bf16", window=32, k=2)
    return [
        # the smallest call: one 512-token layer of the tiny fp32 geometry
        dict(name="step_512_fp32", kind="step", hq=4, hkv=2, d=64, dtype="f32", window=8, k=2,
             batch=1, lo=512, hi=512, budget=64, pool=5, plant=True),
        # an ordinary prompt, evicted layer by layer
        dict(name="step_4096", kind="step", **llama, batch=1, lo=4096, hi=4096, budget=512,
             pool=7, plant=True),
        # one 16K prompt, all 32 layers scored by one call after drafting
        dict(name="score_16k_32_layers", kind="score", **llama, layers=32, batch=1, lo=16384,
             hi=16384, rows="window_draft", lse=False, plant=True),
        # the same cache scored by the draft rows alone (the paper's own scorer)
        dict(name="score_draft_16k_32_layers", kind="score", **llama, layers=32, batch=1,
             lo=16384, hi=16384, rows="draft", lse=False, plant=True),
        # the serving batch: eight ragged sequences of 16K-32K, all 32 layers
        dict(name="score_batch8_32_layers", kind="score", **llama, layers=32, batch=8, lo=16384,
             hi=32768, rows="window_draft", lse=False, plant=False),
        # an engine whose attention forward returns the rows' log-sum-exp; odd lengths
        dict(name="score_lse_ragged_16_layers", kind="score", **llama, layers=16, batch=3,
             lo=5003, hi=12289, rows="window_draft", lse=True, plant=True),
        # selection and compaction of the serving batch
        dict(name="select_batch8_32_layers", kind="select", **llama, layers=32, batch=8, lo=16384,
             hi=32768, budget_first=2048, budget_last=2048, pool=7),
        # H2O over an 8K prompt, everything computed here
        dict(name="h2o_8k", kind="h2o", hq=32, hkv=8, d=128, dtype="bf16", window=0, k=2, batch=1,
             lo=8192, hi=8192, lse=False),
        # H2O of a ragged batch with the log-sum-exp of the prefill
        dict(name="h2o_lse_ragged", kind="h2o", hq=32, hkv=8, d=128, dtype="bf16", window=0, k=2,
             batch=3, lo=1777, hi=4801, lse=True),
        # the scoring rows of one layer through the fused W_q, W_k
        dict(name="project_34_rows", kind="project", n_rows=34, hidden=4096, heads=40, d=128),
        # every row of an 8K prompt through W_q
        dict(name="project_8194_rows", kind="project", n_rows=8194, hidden=4096, heads=32, d=128),
        # diagnostics of the serving batch's compacted cache, one layer
        dict(name="attend_batch8", kind="attend", **llama, batch=8, n_select=2016, n_q=34),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["step", "score", "score", "select", "h2o", "project", "attend"])
    if kind == "project":
        few = rng.random() < 0.5
        return dict(kind=kind, n_rows=_log_int(rng, 2, 64) if few else _log_int(rng, 65, 8194),
                    hidden=128 * _log_int(rng, 8, 32), heads=rng.choice([8, 32, 40]),
                    d=rng.choice([64, 128, 128]))
    if kind == "h2o":
        lo = _log_int(rng, 256, 6000)
        return dict(kind=kind, hq=rng.choice([8, 16, 32]), hkv=8, d=128, dtype="bf16", window=0,
                    k=rng.randint(1, 8), batch=rng.randint(1, 2), lo=lo,
                    hi=lo + rng.randint(0, lo // 3), lse=rng.random() < 0.5)
    geom = dict(hq=rng.choice([8, 16, 32, 32, 32]), hkv=8, d=rng.choice([64, 128, 128, 128]),
                dtype="bf16", window=rng.choice([8, 16, 32, 32]), k=rng.randint(1, 8))
    if kind == "attend":
        tail = geom["window"] + geom["k"]
        return dict(kind=kind, **geom, batch=rng.randint(1, 8), n_select=_log_int(rng, 32, 2048),
                    n_q=rng.choice([1, geom["k"], tail]))
    if kind == "step":
        if rng.random() < 0.25:
            geom.update(dtype="f32")
        lo = _log_int(rng, 300, 12000)
        batch = rng.randint(1, 2)
        return dict(kind=kind, **geom, batch=batch, lo=lo,
                    hi=lo + (rng.randint(0, lo // 3) if batch > 1 else 0),
                    budget=geom["window"] + _log_int(rng, 24, max(25, lo // 4)),
                    pool=rng.choice([1, 5, 7]), plant=True)
    layers, batch = _log_int(rng, 1, 32), rng.randint(1, 4)
    lo = _log_int(rng, 1000, 16384)
    hi = lo + (rng.randint(0, lo) if batch > 1 else 0)
    if kind == "score":
        return dict(kind=kind, **geom, layers=layers, batch=batch, lo=lo, hi=hi,
                    rows=rng.choice(["window_draft", "window_draft", "draft", "window"]),
                    lse=rng.random() < 0.3, plant=rng.random() < 0.5)
    first = geom["window"] + _log_int(rng, 64, 2048)
    return dict(kind=kind, **geom, layers=layers, batch=batch, lo=lo, hi=hi, budget_first=first,
                budget_last=geom["window"] + _log_int(rng, 32, first - geom["window"]),
                pool=rng.choice([1, 5, 7]))


# ---------------------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------------------
def _lens(c):
    """Cached rows of each sequence: prompt lengths spread over [lo, hi], and k draft rows."""
    n = [c["lo"] + int((c["hi"] - c["lo"]) * ((0.5 + 0.6180339887 * b) % 1.0))
         for b in range(c["batch"])]
    return [x + c["k"] for x in n]


def _n_rows(c):
    return {"window_draft": c["window"] + c["k"], "draft": c["k"], "window": c["window"]}[c["rows"]]


def _first_pos(c):
    """The first scoring row's distance from the end of its sequence."""
    return {"window_draft": c["window"] + c["k"], "draft": c["k"],
            "window": c["window"] + c["k"]}[c["rows"]]


def _elt(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _budgets(c):
    nl = c["layers"]
    return [round(c["budget_first"] + (c["budget_last"] - c["budget_first"]) * l / max(nl - 1, 1))
            for l in range(nl)]


def _geometry(c, layers=1):
    return dge.Geometry(c["hq"] * layers, c["hkv"] * layers, c["d"], c["window"], c["k"],
                        [int(x) for x in _lens(c)],
                        dtype=dge.DGE_BF16 if c["dtype"] == "bf16" else dge.DGE_F32, device=DEV)


def work(c):
    if c["kind"] == "project":
        cols = c["heads"] * c["d"]
        return {"bytes": 2 * (c["n_rows"] * (c["hidden"] + cols) + cols * c["hidden"]),
                "flops": 2 * c["n_rows"] * c["hidden"] * cols}
    e = 2 if c["dtype"] == "bf16" else 4
    row = c["d"] * e
    if c["kind"] == "attend":
        tail = c["window"] + c["k"]
        rows = c["batch"] * c["n_q"]
        kv = c["batch"] * c["hkv"] * (c["n_select"] + tail) * row
        mass = c["n_q"] <= tail and c["n_q"] > 1
        vis = c["n_select"] + (tail if not mass else (tail + 1) / 2)
        fl = 2 * c["hq"] * rows * vis * c["d"]
        return {"bytes": 2 * kv + c["hq"] * rows * (row + 4 * c["d"] + 12), "flops": 2 * fl}
    n = _lens(c)
    T = sum(n)
    if c["kind"] == "h2o":
        return {"bytes": T * (c["hkv"] * (row + 4) + c["hq"] * (row + (4 if c["lse"] else 0))),
                "flops": 2 * c["hq"] * c["d"] * sum(x * (x + 1) / 2 for x in n)}
    if c["kind"] == "select":
        out = sum(c["batch"] * c["hkv"] * (4 * (b - c["window"])
                  + 4 * row * (b + c["k"])) for b in _budgets(c))
        return {"bytes": 4 * c["layers"] * c["hkv"] * T + out, "flops": 0}
    nl = c.get("layers", 1)
    nr = _n_rows(c) if c["kind"] == "score" else c["window"] + c["k"]
    b = nl * (c["hkv"] * T * (row + 4) + c["hq"] * c["batch"] * nr * (row + (4 if c.get("lse") else 0)))
    if c["kind"] == "step":
        b += c["batch"] * c["hkv"] * (4 * (c["budget"] - c["window"]) + 4 * row * (c["budget"] + c["k"]))
    return {"bytes": b, "flops": 2 * nl * c["hq"] * nr * T * c["d"]}


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(0x5EED0000 + int(seed))
    return g


def _normal(g, shape, dtype):
    """Standard normal values; leading slices are drawn one by one to bound temporaries."""
    x = torch.empty(shape, dtype=dtype, device=DEV)
    flat = x.view(-1, x.shape[-1])
    step = max(1, (1 << 28) // x.shape[-1])
    for i in range(0, flat.shape[0], step):
        part = flat[i:i + step]
        part.copy_(torch.randn(part.shape, generator=g, device=DEV))
    return x


def _plant(g, c, q, k, n_rows):
    """Spans of 16 keys in every KV head pulled by 4 sqrt(d) along the group's mean query."""
    H, d = k.shape[0], c["d"]
    s0 = 0
    for b, n in enumerate(_lens(c)):
        cand = n - c["window"] - c["k"]
        slots = cand // 32
        spans = min(math.ceil(0.01 * (n - c["k"]) / 16), slots)
        if spans > 0:
            u = q[:, b * n_rows:(b + 1) * n_rows].float().reshape(H, -1, d).mean(1)
            u = 4 * math.sqrt(d) * u / u.norm(dim=1, keepdim=True)
            slot = torch.rand(H, slots, generator=g, device=DEV).argsort(1)[:, :spans]
            start = slot * 32 + torch.randint(0, 17, (H, spans), generator=g, device=DEV)
            rows = (s0 + start[:, :, None] + torch.arange(16, device=DEV)).reshape(H, -1)
            at = rows[:, :, None].expand(-1, -1, d)
            k.scatter_(1, at, (k.gather(1, at).float() + u[:, None]).to(k.dtype))
        s0 += n


def _visible(c, n_q, kept):
    """Rows of the compacted cache that each of the n_q query rows attends."""
    tail = c["window"] + c["k"]
    from_end = n_q if n_q > 1 else 0
    return [kept + (tail if from_end == 0 else tail - from_end + r + 1) for r in range(n_q)]


def _kept(c):
    """Retained past keys of each sequence: the budget, and less in one short sequence."""
    return [c["n_select"] if b != 1 else max(1, c["n_select"] * 3 // 4) for b in range(c["batch"])]


def prepare(case, seed):
    c = dict(case)
    g = _generator(seed)
    s = {"case": c}
    if c["kind"] == "project":
        cols = c["heads"] * c["d"]
        s["x"] = _normal(g, (c["n_rows"], c["hidden"]), torch.bfloat16)
        s["w"] = (torch.randn(cols, c["hidden"], generator=g, device=DEV)
                  / math.sqrt(c["hidden"])).to(torch.bfloat16)
        first = int(torch.randint(0, 16384, (1,), generator=g, device=DEV))
        s["positions"] = torch.arange(first, first + c["n_rows"], dtype=torch.int32, device=DEV)
        return s
    if c["kind"] == "attend":
        tail = c["window"] + c["k"]
        c.update(lo=4 * c["n_select"] + tail, hi=4 * c["n_select"] + tail)
        s["geom"] = _geometry(c)
        shape = (c["batch"], c["hkv"], c["n_select"] + tail, c["d"])
        s["q"] = _normal(g, (c["hq"], c["batch"] * c["n_q"], c["d"]), _elt(c))
        s["k_c"], s["v_c"] = _normal(g, shape, _elt(c)), _normal(g, shape, _elt(c))
        s["n_kept"] = torch.zeros(max(c["batch"], 4), dtype=torch.int32, device=DEV)
        s["n_kept"][:c["batch"]] = torch.tensor(_kept(c), dtype=torch.int32)
        if c["n_q"] > 1:
            # full-cache partitions: the retained keys' and a share of mass on evicted ones
            lse = _attend64(c, s["q"], s["k_c"], None)[1]
            lost = 0.05 + 0.75 * torch.rand(lse.shape, generator=g, device=DEV, dtype=torch.float64)
            s["lse_full"] = (lse - torch.log1p(-lost)).float()
        return s
    n = _lens(c)
    T = sum(n)
    if c["kind"] == "h2o":
        s["geom"] = _geometry(c)
        s["q"] = _normal(g, (c["hq"], T, c["d"]), _elt(c))
        s["key"] = _normal(g, (c["hkv"], T, c["d"]), _elt(c))
        s["lse"] = _h2o64(c, s["q"], s["key"])[1].float() if c["lse"] else None
        s["ws"] = torch.empty(dge.workspace_size(s["geom"], dge.OP_H2O), dtype=torch.uint8, device=DEV)
        return s
    if c["kind"] == "select":
        nl = c["layers"]
        s["geom"] = _geometry(c)
        s["n_select"] = [b - c["window"] for b in _budgets(c)]
        s["scores"] = torch.empty(nl * c["hkv"], T, device=DEV)
        for l in range(nl):
            x = torch.zeros(c["hkv"], T, device=DEV)
            for _ in range(8):
                x += torch.randn(x.shape, generator=g, device=DEV).exp_()
            s["scores"][l * c["hkv"]:(l + 1) * c["hkv"]] = x * (4.25 / T)
        s["key"] = _normal(g, (nl * c["hkv"], T, c["d"]), _elt(c))
        s["value"] = _normal(g, (nl * c["hkv"], T, c["d"]), _elt(c))
        heads, tail = c["batch"] * c["hkv"], c["window"] + c["k"]
        rows = heads * sum(x + tail for x in s["n_select"])
        s["idx"] = torch.empty(max(heads * sum(s["n_select"]), 4), dtype=torch.int32, device=DEV)
        s["k_out"] = torch.empty(rows, c["d"], dtype=_elt(c), device=DEV)
        s["v_out"] = torch.empty(rows, c["d"], dtype=_elt(c), device=DEV)
        s["ws"] = torch.empty(dge.workspace_size(s["geom"], dge.OP_SELECT), dtype=torch.uint8, device=DEV)
        return s
    nl = c.get("layers", 1)
    if c["kind"] == "step":
        c["rows"] = "window_draft"
    nr = _n_rows(c)
    s["geom"] = _geometry(c, nl)
    s["q"] = _normal(g, (nl * c["hq"], c["batch"] * nr, c["d"]), _elt(c))
    s["key"] = _normal(g, (nl * c["hkv"], T, c["d"]), _elt(c))
    if c["plant"]:
        _plant(g, c, s["q"], s["key"], nr)
    if c["kind"] == "step":
        s["value"] = _normal(g, (nl * c["hkv"], T, c["d"]), _elt(c))
        return s
    s["raw"] = torch.empty(nl * c["hkv"], T, device=DEV)
    if c["lse"]:
        s["lse"] = _score64(c, s["q"], s["key"], False)[1].float()
    else:
        s["ws"] = torch.empty(dge.workspace_size(s["geom"], dge.OP_SCORE), dtype=torch.uint8, device=DEV)
    return s


# ---------------------------------------------------------------------------------------
# the timed calls
# ---------------------------------------------------------------------------------------
def run(s):
    c = s["case"]
    if c["kind"] == "step":
        return dge.evict_layer(s["geom"], s["q"], s["key"], s["value"], c["budget"], c["pool"])
    if c["kind"] == "score":
        if c["lse"]:
            return {"raw": dge.score_lse(s["geom"], ROWS[c["rows"]], s["q"], s["key"], s["lse"],
                                         raw=s["raw"])}
        return {"raw": dge.score(s["geom"], ROWS[c["rows"]], s["q"], s["key"], raw=s["raw"],
                                 ws=s["ws"])}
    if c["kind"] == "select":
        n_kept = dge.select_compact_layers(s["geom"], s["scores"], c["pool"], c["window"] + c["k"],
                                           s["n_select"], s["key"], s["value"], idx=s["idx"],
                                           k_out=s["k_out"], v_out=s["v_out"], ws=s["ws"])[1]
        return {"idx": s["idx"], "n_kept": n_kept, "k": s["k_out"], "v": s["v_out"]}
    if c["kind"] == "h2o":
        return {"colsum": dge.h2o_colsum(s["geom"], s["q"], s["key"], lse=s["lse"], ws=s["ws"])}
    if c["kind"] == "project":
        return {"out": dge.project_rope(s["x"], s["w"], s["positions"], c["heads"], c["d"])}
    tail = c["window"] + c["k"]
    from_end = c["n_q"] if c["n_q"] > 1 else 0
    out, lse = dge.cache_attention(s["geom"], s["q"], c["n_q"], from_end, s["k_c"], s["v_c"],
                                   c["n_select"], tail, s["n_kept"])
    if c["n_q"] == 1:
        return {"out": out, "lse": lse}
    rho, beta, l_match = dge.evicted_mass(s["geom"], s["q"], c["n_q"], from_end, s["k_c"],
                                          c["n_select"], tail, s["n_kept"], s["lse_full"])
    return {"out": out, "lse": lse, "rho": rho, "beta": beta, "l_match": l_match}


# ---------------------------------------------------------------------------------------
# the same results in 64 bits, with plain torch
# ---------------------------------------------------------------------------------------
def _score64(c, q, k, columns=True):
    """Column sums (or None) and row log-sum-exps of the scoring rows."""
    nr, G, n = _n_rows(c), c["hq"] // c["hkv"], _lens(c)
    H, T = k.shape[0], k.shape[1]
    raw = torch.empty(H, T, dtype=torch.float64, device=DEV) if columns else None
    lse = torch.empty(q.shape[0], q.shape[1], dtype=torch.float64, device=DEV)
    s0 = 0
    for b, N in enumerate(n):
        pos = (N - _first_pos(c) + torch.arange(nr, device=DEV)).repeat(G)
        lo = N - _first_pos(c)
        hidden = torch.arange(lo, N, device=DEV)[None] > pos[:, None]
        for h in range(H):
            qr = q[h * G:(h + 1) * G, b * nr:(b + 1) * nr].reshape(G * nr, -1).double()
            x = qr @ k[h, s0:s0 + N].double().T.contiguous() / math.sqrt(c["d"])
            x[:, lo:].masked_fill_(hidden, -math.inf)
            z = torch.logsumexp(x, 1)
            lse[h * G:(h + 1) * G, b * nr:(b + 1) * nr] = z.view(G, nr)
            if columns:
                raw[h, s0:s0 + N] = (x - z[:, None]).exp_().sum(0) / G
        s0 += N
    return raw, lse


def _h2o64(c, q, k):
    G, H, T = c["hq"] // c["hkv"], c["hkv"], k.shape[1]
    col = torch.zeros(H, T, dtype=torch.float64, device=DEV)
    lse = torch.empty(c["hq"], T, dtype=torch.float64, device=DEV)
    s0 = 0
    for N in _lens(c):
        for hq in range(c["hq"]):
            kt = k[hq // G, s0:s0 + N].double().T.contiguous()
            for r0 in range(0, N, 2048):  # row blocks bound the memory
                r1 = min(N, r0 + 2048)
                x = q[hq, s0 + r0:s0 + r1].double() @ kt[:, :r1].contiguous() / math.sqrt(c["d"])
                hidden = (torch.arange(r1, device=DEV)[None] > torch.arange(r0, r1, device=DEV)[:, None])
                x.masked_fill_(hidden, -math.inf)
                z = torch.logsumexp(x, 1)
                lse[hq, s0 + r0:s0 + r1] = z
                col[hq // G, s0:s0 + r1] += (x - z[:, None]).exp_().sum(0) / G
        s0 += N
    return col, lse


def _attend64(c, q, k_c, v_c):
    """Outputs (None without v_c) and log-partitions over the compacted caches."""
    G, n_q = c["hq"] // c["hkv"], c["n_q"]
    out = None if v_c is None else torch.empty(q.shape, dtype=torch.float64, device=DEV)
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device=DEV)
    for b, kept in enumerate(_kept(c)):
        vis = torch.tensor(_visible(c, n_q, kept), device=DEV).repeat(G)
        for h in range(c["hkv"]):
            qr = q[h * G:(h + 1) * G, b * n_q:(b + 1) * n_q].reshape(G * n_q, -1).double()
            x = qr @ k_c[b, h].double().T.contiguous() / math.sqrt(c["d"])
            x.masked_fill_(torch.arange(x.shape[1], device=DEV)[None] >= vis[:, None], -math.inf)
            z = torch.logsumexp(x, 1)
            lse[h * G:(h + 1) * G, b * n_q:(b + 1) * n_q] = z.view(G, n_q)
            if v_c is not None:
                o = (x - z[:, None]).exp_() @ v_c[b, h].double()
                out[h * G:(h + 1) * G, b * n_q:(b + 1) * n_q] = o.view(G, n_q, -1)
    return out, lse


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "select":
        return None  # indices and copies
    s = prepare(case, seed)
    if c["kind"] == "project":
        y = (s["x"].double() @ s["w"].double().T.contiguous()).view(c["n_rows"], c["heads"], c["d"])
        half = c["d"] // 2
        freq = 500000.0 ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / c["d"])
        a = (s["positions"].double()[:, None] * freq)[:, None]
        lo, hi = y[..., :half], y[..., half:]
        y = torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)
        return {"out": y.transpose(0, 1).contiguous()}
    if c["kind"] == "attend":
        out, lse = _attend64(c, s["q"], s["k_c"], s["v_c"])
        if c["n_q"] == 1:
            return {"out": out, "lse": lse}
        lost = (s["lse_full"].double() - lse).clamp_min(0)
        rho = -torch.expm1(-lost)
        per = (c["hkv"], c["hq"] // c["hkv"], c["batch"], c["n_q"])
        return {"out": out, "lse": lse, "rho": rho,
                "beta": rho.view(per).mean((1, 3)).T.contiguous(),
                "l_match": lost.view(per).mean((1, 3)).T.contiguous()}
    if c["kind"] == "h2o":
        return {"colsum": _h2o64(c, s["q"], s["key"])[0]}
    c.setdefault("rows", "window_draft")
    raw = _score64(c, s["q"], s["key"])[0]
    return {"raw": raw} if c["kind"] == "score" else {"raw": raw, "idx": None, "n_kept": None,
                                                      "k": None, "v": None}


def tolerance(c):
    # About four times what the results differ by from 64-bit sums (measured: scores and
    # column sums 0.2 to 1.0e-6, attention outputs 1e-5, whose weights enter the product in
    # two bf16 parts).  The query capture rounds once to bf16: two correct sums differ in
    # the rounding of a few values by one unit in the last place (2^-8 to 2^-7 of the value).
    if c["kind"] == "select":
        return "exact"  # given scores, the selection is a rule and the rows are copies
    if c["kind"] == "project":
        return {"rel": 2e-3, "max": 1.6e-2}
    if c["kind"] == "attend":
        return {"rel": 4e-5, "max": 1e-3}
    if c["kind"] == "step":  # a key at the threshold may swap with the next one
        return {"rel": 5e-6, "max": 2e-4, "differ": 2e-3}
    return {"rel": 5e-6, "max": 2e-4}
