"""The work that is timed: calls of the retention step and of its decode-side consumer through
``paper_2602_08686_amd.binding``, over the range of shapes its users have.

``listed()`` names the cases, ``draw(rng)`` gives another one of the same ranges, ``prepare`` makes what a
program has in hand before the call, ``run`` is one pass, ``work`` what a pass cannot do without,
``tolerance`` how far two correct results may be apart, ``exact`` the same results in 64 bits from plain
torch (results that an integer decision makes -- index lists, counts, and the rows copied by them -- have no
64-bit counterpart and are left out).

Four kinds of case:
  layer    one layer's whole step: scan, tables, selection, gather (with the scan and the tables as one call,
           as bench.py does, or as separate calls), optionally with the value-norm factor, with the risk gate,
           with normalisers that the prefill's attention kernel left
  keep     selection and gather on utilities that a caller already has
  shared   the layer-shared mode over a few layers: one alpha and one index list per layer for all heads
  decode   attention of decoding queries over a ragged compact cache, or over a full one
"""
import math

import torch

from paper_2602_08686_amd import binding as B
from paper_2602_08686_amd import workloads as wl

POOLS = {"none": wl.POOL_NONE, "avg": wl.POOL_AVG, "max": wl.POOL_MAX}


def _layer(name, dtype, batch, q_heads, kv_heads, d, length, window, pool, kernel, budget, **kw):
    c = {"kind": "layer", "dtype": dtype, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "d": d, "length": length,
         "window": window, "pool": pool, "kernel": kernel, "budget": budget, "one_call": True, "value_norm": False,
         "given_lse": False, "shares": False, "gate": False, "keys": "plain"}
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest: one short f32 prompt, the separate calls; launches and latency
        _layer("layer_f32_1k", "f32", 1, 4, 4, 64, 1024, 32, "avg", 7, 128, one_call=False, shares=True, keys="needles"),
        # a chat-length prompt of a model without grouped queries, with an attention sink
        _layer("layer_mha_4k", "bf16", 1, 32, 32, 128, 4096, 32, "max", 7, 512, keys="sink"),
        # a prompt whose length is no round number (most prompts): batch 2, 20011 tokens
        _layer("layer_ragged_20k", "bf16", 2, 32, 8, 128, 20011, 32, "avg", 7, 512, shares=True, keys="pareto"),
        # batch serving at 32k, the shape the benchmark is quoted on: the largest
        _layer("layer_gqa_32k_b16", "bf16", 16, 32, 8, 128, 32768, 32, "avg", 7, 512, shares=True, keys="pareto"),
        # a single very long prompt with a wide observation window
        _layer("layer_gqa_128k_w64", "bf16", 1, 32, 8, 128, 131072, 64, "max", 7, 512, shares=True, keys="needles"),
        # groups of seven query heads, scale-biased heads, the risk gate
        _layer("layer_g7_64k", "bf16", 4, 28, 4, 128, 65536, 32, "avg", 5, 1024, gate=True, keys="scaled"),
        # the value-norm factor, separate calls, a ragged length
        _layer("layer_vnorm_10k", "bf16", 4, 32, 8, 128, 10006, 32, "avg", 7, 256, one_call=False, value_norm=True, shares=True),
        # the prefill's attention kernel already has the window rows' normalisers: one pass over K
        _layer("layer_lse_16k", "bf16", 4, 32, 8, 128, 16384, 32, "avg", 7, 256, given_lse=True, shares=True, keys="pareto"),
        # selection and gather alone, a length that is no multiple of four
        {"name": "keep_50k", "kind": "keep", "dtype": "bf16", "batch": 2, "kv_heads": 8, "d": 128, "length": 50001, "window": 32,
         "budget": 1024},
        # the paper's Alg. 1 as printed, over four layers
        {"name": "shared_16k", "kind": "shared", "dtype": "bf16", "batch": 4, "q_heads": 32, "kv_heads": 8, "d": 128,
         "length": 16384, "window": 32, "budget": 256, "layers": 4},
        # one layer of a decoding step over the compact cache of a batch of 32k prompts
        {"name": "decode_compact", "kind": "decode", "dtype": "bf16", "batch": 16, "q_heads": 32, "kv_heads": 8, "d": 128,
         "rows": 544, "queries": 1, "ragged": True},
        # the same over an uncompressed cache (what the discarded mass is measured against)
        {"name": "decode_full_32k", "kind": "decode", "dtype": "bf16", "batch": 4, "q_heads": 32, "kv_heads": 8, "d": 128,
         "rows": 32768, "queries": 1, "ragged": False},
    ]


# what bounds the cost of a drawn case: the bytes of K, and heads x 32-row tiles x keys, of the largest listed one
MOST_K = 16 * 8 * 32768 * 128 * 2
MOST_TILES = 16 * 32 * 32768


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _length(rng, lo, hi):
    """Lengths over the logarithm of the range: two in three as they come, one in three a round number."""
    n = _log_uniform(rng, lo, hi)
    return n if rng.random() < 2 / 3 else max(lo, n // 512 * 512)


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["keep", "shared", "decode", "decode"])
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    e = 4 if dtype == "f32" else 2
    kv, group = rng.choice([(8, 4), (8, 4), (4, 7), (32, 1), (8, 1), (8, 2), (4, 8), (2, 6), (1, 8), (8, 5)])
    d = rng.choice([128, 128, 128, 64])
    if kind == "layer":
        n = _length(rng, 512, 131072 if dtype == "bf16" else 16384)
        window = rng.choice([32, 32, 32, 64, 16, 48])
        # products of 32 x 32 query rows and keys, f32 ones counted as they take the matrix cores longer
        tiles = kv * group * ((window + 31) // 32) * d / 128 * (8 if dtype == "f32" else 1)
        n = min(n, int(MOST_TILES / tiles))
        batch = min(_log_uniform(rng, 1, 16), max(1, MOST_K // (2 * kv * n * d * e)), max(1, int(MOST_TILES / (tiles * n))))
        pool = rng.choice(["avg", "avg", "max", "none"])
        c = _layer(None, dtype, batch, kv * group, kv, d, n, window, pool, 1 if pool == "none" else rng.choice([3, 5, 7, 7, 9, 13]),
                   min(max(window + 32, rng.choice([128, 256, 512, 1024, 2048])), max(window + 32, n // 8)))
        c.update(one_call=rng.random() < 0.75, value_norm=rng.random() < 0.25, given_lse=rng.random() < 0.25,
                 shares=rng.random() < 0.5, gate=rng.random() < 0.25,
                 keys=rng.choice(["plain", "pareto", "sink", "needles", "scaled"]))
        return c
    if kind == "keep":
        n = _length(rng, 1024, 131072)
        return {"kind": "keep", "dtype": dtype, "batch": min(_log_uniform(rng, 1, 16), max(1, MOST_K // (kv * n * d * e))),
                "kv_heads": kv, "d": d, "length": n, "window": 32, "budget": min(rng.choice([128, 512, 1024, 2048]), n // 4)}
    if kind == "shared":
        layers = rng.choice([2, 4])
        n = _length(rng, 1024, 32768)
        return {"kind": "shared", "dtype": "bf16", "batch": min(_log_uniform(rng, 1, 8), max(1, MOST_K // (4 * layers * kv * n * d * e))),
                "q_heads": kv * group, "kv_heads": kv, "d": d, "length": n, "window": 32, "budget": min(512, n // 4), "layers": layers}
    compact = rng.random() < 0.6
    n = _log_uniform(rng, 96, 4096) if compact else _length(rng, 4097, 131072)
    queries = rng.choice([1, 1, 1, 2, 4])
    batch = min(_log_uniform(rng, 1, 32), max(1, MOST_K // (2 * kv * n * d * e * queries)))
    return {"kind": "decode", "dtype": dtype, "batch": batch, "q_heads": kv * group, "kv_heads": kv, "d": d, "rows": n,
            "queries": queries, "ragged": compact}


# ---------------------------------------------------------------------------------------------------------
def _workload(c, seed, **kw):
    keys = c.get("keys", "plain")
    return wl.Workload("case", c["dtype"], c["batch"], c["q_heads"], c["kv_heads"], c["d"], c["length"], c["window"],
                       POOLS[c.get("pool", "none")], c.get("kernel", 1), c["budget"], c.get("layers", 1), seed=seed,
                       needles=16 if keys == "needles" else 0, sink_scale=8.0 if keys in ("sink", "needles") else 0.0,
                       pareto_frac=0.05 if keys == "pareto" else 0.0, head_key_scale=keys == "scaled",
                       shares=c.get("shares", False), gate=c.get("gate", False), **kw)


def _window_lse(q, k, scale):
    """Normalisers of the window rows as an attention kernel leaves them: fp32, natural log, causal."""
    batch, hq, w, _ = q.shape
    kv, length = k.shape[1], k.shape[2]
    out = torch.empty(batch, hq, w, device=q.device)
    mask = torch.ones(w, length, dtype=torch.bool, device=q.device).tril(length - w)
    for b in range(batch):
        for h in range(hq):
            z = (q[b, h].float() @ k[b, h // (hq // kv)].float().t()) * scale
            out[b, h] = torch.logsumexp(z.masked_fill_(~mask, -math.inf), 1)
    return out


def prepare(case, seed):
    c = case
    if c["kind"] == "layer":
        w = _workload(c, seed)
        t, tables = wl.make_layer(w, 0, "cuda"), wl.make_tables(w, "cuda")
        p = B.params_for(t["q"], t["k"], t["v"], pool=w.pool, pool_kernel=w.pool_kernel, budget=w.budget, cap=w.cap,
                         n_layers=w.n_layers, flags=B.FLAG_VALUE_NORM if c["value_norm"] else 0)
        lse = _window_lse(t["q"], t["k"], 1.0 / math.sqrt(w.head_dim)) if c["given_lse"] else None
        return {"case": c, "p": p, "t": t, "tables": tables, "lse": lse, "buf": B.LayerBuffers(p, "cuda")}
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7919 + 17)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    if c["kind"] == "keep":
        batch, kv, n, d, win = c["batch"], c["kv_heads"], c["length"], c["d"], c["window"]
        k = torch.randn(batch, kv, n, d, generator=g, device="cuda").to(dt)
        v = torch.randn(batch, kv, n, d, generator=g, device="cuda").to(dt)
        # masses of a softmax over near-normal logits are log-normal; a few tokens stand far out
        u = torch.randn(batch, kv, n - win, generator=g, device="cuda").mul_(0.6).exp_()
        u[..., :4] *= 50.0
        budget = torch.randint(win, c["budget"] + 1, (batch, kv), generator=g, device="cuda", dtype=torch.int32)
        cap = min(n, c["budget"] * kv - (kv - 1) * win)  # rows of an index list, as the call's rule has it
        p = B.make_params(batch=batch, n_q_heads=kv, n_kv_heads=kv, head_dim=d, seq_len=n, window=win, dtype=dt,
                          pool=wl.POOL_NONE, pool_kernel=1, budget=c["budget"], cap=cap)
        return {"case": c, "p": p, "k": k, "v": v, "u": u, "budget": budget, "tau": torch.zeros(batch, device="cuda"),
                "idx": torch.full((batch, kv, cap), -1, dtype=torch.int32, device="cuda"),
                "count": torch.empty(batch, kv, dtype=torch.int32, device="cuda"),
                "k_out": torch.zeros(batch, kv, cap, d, dtype=dt, device="cuda"),
                "v_out": torch.zeros(batch, kv, cap, d, dtype=dt, device="cuda"),
                "ws": torch.empty(max(B.ckv_workspace_bytes(p), 256), dtype=torch.uint8, device="cuda")}
    if c["kind"] == "shared":
        w = _workload(dict(c, gate=True, keys="pareto"), seed)
        layers, tables = [wl.make_layer(w, i, "cuda") for i in range(w.n_layers)], wl.make_tables(w, "cuda")
        flags = B.FLAG_VALUE_NORM | (B.FLAG_GROUP_MASS if w.window <= 32 and w.group <= 4 else 0)
        ps = [B.params_for(t["q"], t["k"], t["v"], pool=w.pool, pool_kernel=w.pool_kernel, budget=w.budget, cap=w.cap, layer=i,
                           n_layers=w.n_layers, flags=flags) for i, t in enumerate(layers)]
        one = B.make_params(batch=w.batch, n_q_heads=1, n_kv_heads=1, head_dim=w.head_dim, seq_len=w.seq_len, window=w.window,
                            dtype=w.dtype, pool=wl.POOL_NONE, pool_kernel=1, budget=w.budget, cap=w.cap, n_layers=w.n_layers)
        n, batch, cap = w.n_layers, w.batch, w.cap
        new = lambda *s, dtype=torch.float32: torch.zeros(*s, dtype=dtype, device="cuda")  # noqa: E731
        return {"case": c, "w": w, "layers": layers, "tables": tables, "ps": ps, "one": one, "buf": B.LayerBuffers(ps[0], "cuda"),
                "alpha": new(batch, w.seq_len), "rho": new(n, batch, w.n_kv_heads, w.seq_len), "risk": new(batch),
                "bin": new(batch, dtype=torch.int32), "edges": torch.linspace(0.0, math.log(w.seq_len), 19, device="cuda"),
                "u": new(n, batch, w.prefix), "tau": new(n, batch),
                "budget": torch.full((batch, 1), w.budget, dtype=torch.int32, device="cuda"),
                "idx": new(n, batch, cap, dtype=torch.int32), "count": new(n, batch, dtype=torch.int32),
                "k_out": new(n, batch, w.n_kv_heads, cap, w.head_dim, dtype=w.torch_dtype),
                "v_out": new(n, batch, w.n_kv_heads, cap, w.head_dim, dtype=w.torch_dtype)}
    batch, hq, kv, d, n, nq = c["batch"], c["q_heads"], c["kv_heads"], c["d"], c["rows"], c["queries"]
    k = torch.randn(batch, kv, n, d, generator=g, device="cuda").to(dt)
    v = torch.randn(batch, kv, n, d, generator=g, device="cuda").to(dt)
    q = torch.randn(batch, hq, nq, d, generator=g, device="cuda").to(dt)
    count = torch.randint(max(1, n // 2), n + 1, (batch, kv), generator=g, device="cuda", dtype=torch.int32) if c["ragged"] else None
    p = B.make_params(batch=batch, n_q_heads=hq, n_kv_heads=kv, head_dim=d, seq_len=n, window=min(32, n), dtype=dt,
                      pool=wl.POOL_NONE, pool_kernel=1, budget=n, cap=n)
    return {"case": c, "p": p, "k": k, "v": v, "q": q, "count": count, "out": torch.empty(batch, hq, nq, d, device="cuda"),
            "lse": torch.empty(batch, hq, nq, device="cuda"),
            "ws": torch.empty(max(B.ckv_decode_workspace_bytes(p, nq, n), 256), dtype=torch.uint8, device="cuda")}


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "layer":
        t, buf = s["t"], s["buf"]
        B.retention_layer(s["p"], t["q"], t["k"], t["v"], s["tables"], buf, lse=s["lse"], fused_utility=s["case"]["one_call"])
        out = {"utility": buf.utility, "tau": buf.tau, "budget": buf.budget, "idx": buf.idx, "count": buf.count,
               "k_out": buf.k_out, "v_out": buf.v_out}
        if not s["case"]["one_call"]:
            out["scores"] = buf.scores
        if buf.vnorm_ratio is not None:
            out["rho"] = buf.vnorm_ratio
        return out
    if kind == "keep":
        B.ckv_select_topk(s["p"], s["u"], s["budget"], s["tau"], s["idx"], s["count"], s["ws"])
        B.ckv_compact_kv(s["p"], s["k"], s["v"], s["idx"], s["count"], s["k_out"], s["v_out"])
        return {n: s[n] for n in ("idx", "count", "k_out", "v_out")}
    if kind == "shared":
        buf, tables, w = s["buf"], s["tables"], s["w"]
        bins = tables["risk_bins"]
        s["alpha"].zero_()
        for i, t in enumerate(s["layers"]):
            B.ckv_window_scores(s["ps"][i], t["q"], t["k"], t["v"], None, buf.scores, s["rho"][i], buf.workspace)
            B.ckv_alpha_accumulate(s["ps"][i], buf.scores, 1.0 / (w.n_layers * w.n_q_heads), s["alpha"])
        B.ckv_risk_struct(s["ps"][0], s["alpha"], s["edges"], s["risk"], s["bin"])
        bins[:, 0] = s["bin"]
        for i, t in enumerate(s["layers"]):
            B.ckv_shared_utility(s["ps"][i], s["alpha"], s["rho"][i], tables["w_head"], tables["t_gate"], tables["n_ent"],
                                 tables["n_ppl"], bins, s["u"][i], s["tau"][i])
            B.ckv_select_topk(s["one"], s["u"][i], s["budget"], s["tau"][i], s["idx"][i], s["count"][i], buf.workspace)
            B.ckv_compact_kv_shared(s["ps"][i], t["k"], t["v"], s["idx"][i], s["count"][i], s["k_out"][i], s["v_out"][i])
        return {n: s[n] for n in ("alpha", "rho", "risk", "bin", "u", "tau", "idx", "count", "k_out", "v_out")}
    B.ckv_decode_attention(s["p"], s["q"], s["k"], s["v"], s["count"], s["out"], s["lse"], s["ws"])
    return {"out": s["out"], "lse": s["lse"]}


def work(case):
    """Every input byte that the results depend on read once, every output byte written once; one contraction of
    the window's query rows with the keys (with keys and values when decoding)."""
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "decode":
        rows = c["rows"] * (0.75 if c["ragged"] else 1.0)  # ragged: counts are drawn between half and all rows
        per_q = c["batch"] * c["q_heads"] * c["queries"]
        return {"bytes": 2 * c["batch"] * c["kv_heads"] * rows * c["d"] * e + per_q * (c["d"] * (e + 4) + 4),
                "flops": 4.0 * per_q * rows * c["d"]}
    units, n, d, win = c["batch"] * c["kv_heads"], c["length"], c["d"], c["window"]
    k_bytes = units * n * d * e
    if c["kind"] == "keep":
        kept = units * (c["budget"] + win) / 2  # budgets are drawn between the window and the nominal one
        return {"bytes": units * (n - win) * 4 + kept * (4 * d * e + 4) + units * 8, "flops": 0.0}
    q_rows = c["batch"] * c["q_heads"] * win
    scan = k_bytes + q_rows * d * e
    if c["kind"] == "shared":
        kept = c["batch"] * min(c["budget"], n)
        per_layer = scan + k_bytes + units * n * 4 + c["batch"] * (n - win) * 4 + kept * (c["kv_heads"] * 4 * d * e + 4)
        return {"bytes": c["layers"] * per_layer + c["batch"] * n * 4, "flops": c["layers"] * 2.0 * q_rows * n * d}
    kept = units * min(c["budget"], n)
    out = units * (n - win) * 4 + kept * (4 * d * e + 4)
    if c["value_norm"]:
        out += k_bytes + units * n * 4
    if c["given_lse"]:
        out += q_rows * 4
    if not c["one_call"]:
        out += c["batch"] * c["q_heads"] * n * 4
    return {"bytes": scan + out, "flops": 2.0 * q_rows * n * d}


def tolerance(case):
    if case["kind"] == "keep":
        return "exact"  # integers and copied bytes
    if case["kind"] == "decode":
        return {"rel": 2e-6, "max": 4e-5}  # seen against 64 bits: rel 2e-7 to 3e-7
    # logits of a few tens in fp32, so their exponentials carry a few 1e-6: seen against 64 bits, rel 3e-7 to 3.4e-6;
    # no index list differed from the one made with the 64-bit utilities in 1200 (batch, KV head) units
    return {"rel": 1.2e-5, "max": 2e-4}


# ---------------------------------------------------------------------------------------------------------
def _scores64(q, k, b, g, group):
    """Window mass [group, n] of one KV head in 64 bits."""
    win, d = q.shape[2], q.shape[3]
    n = k.shape[2]
    kk = k[b, g].double()
    mask = torch.ones(win, n, dtype=torch.bool, device=q.device).tril(n - win)
    out = torch.empty(group, n, dtype=torch.float64, device=q.device)
    for i in range(group):
        z = (q[b, g * group + i].double() @ kk.t()).mul_(1.0 / math.sqrt(d)).masked_fill_(~mask, -math.inf)
        out[i] = torch.softmax(z, 1).sum(0) * (n / win)
    return out


def _pool64(s, mode, kernel):
    if mode == "none" or kernel == 1:
        return s
    if mode == "avg":
        return torch.nn.functional.avg_pool1d(s[:, None], kernel, 1, kernel // 2, count_include_pad=True)[:, 0]
    return torch.nn.functional.max_pool1d(s[:, None], kernel, 1, kernel // 2)[:, 0]


def _rho64(v):
    r = v.double().norm(dim=-1)
    return r / (r.mean(-1, keepdim=True) + 1e-6)


def exact(case, seed):
    c = case
    if c["kind"] == "keep":
        return None
    s = prepare(c, seed)
    if c["kind"] == "decode":
        batch, hq, kv = c["batch"], c["q_heads"], c["kv_heads"]
        group = hq // kv
        out = torch.empty(batch, hq, c["queries"], c["d"], dtype=torch.float64, device="cuda")
        lse = torch.empty(batch, hq, c["queries"], dtype=torch.float64, device="cuda")
        for b in range(batch):
            for g in range(kv):
                m = c["rows"] if s["count"] is None else int(s["count"][b, g])
                kk, vv = s["k"][b, g, :m].double(), s["v"][b, g, :m].double()
                qq = s["q"][b, g * group:(g + 1) * group].double().reshape(-1, c["d"])
                z = (qq @ kk.t()) / math.sqrt(c["d"])
                lse[b, g * group:(g + 1) * group] = torch.logsumexp(z, 1).view(group, -1)
                out[b, g * group:(g + 1) * group] = (torch.softmax(z, 1) @ vv).view(group, -1, c["d"])
        return {"out": out, "lse": lse}
    batch, kv, n, win = c["batch"], c["kv_heads"], c["length"], c["window"]
    group = c["q_heads"] // kv
    if c["kind"] == "shared":
        w, layers = s["w"], s["layers"]
        alpha = torch.zeros(batch, n, dtype=torch.float64, device="cuda")
        rho = torch.stack([torch.stack([_rho64(t["v"][b]) for b in range(batch)]) for t in layers])
        for t in layers:
            for b in range(batch):
                for g in range(kv):
                    alpha[b] += _scores64(t["q"], t["k"], b, g, group).sum(0) / (w.n_layers * w.n_q_heads)
        a = alpha / alpha.sum(1, keepdim=True)
        wh = s["tables"]["w_head"].double()
        top = wh.view(w.n_layers, kv, group).amax(2)  # alpha and rho are non-negative: the group's largest weight decides
        u = (alpha[None, :, None, :] * rho * top[:, None, :, None]).amax(2)[..., : n - win].contiguous()
        return {"alpha": alpha, "rho": rho, "risk": -torch.special.xlogy(a, a).sum(1), "bin": None, "u": u, "tau": None,
                "idx": None, "count": None, "k_out": None, "v_out": None}
    q, k, v = s["t"]["q"], s["t"]["k"], s["t"]["v"]
    wh = s["tables"]["w_head"][0].double()
    utility = torch.empty(batch, kv, n - win, dtype=torch.float64, device="cuda")
    scores = None if c["one_call"] else torch.empty(batch, c["q_heads"], n, dtype=torch.float64, device="cuda")
    rho = torch.stack([_rho64(v[b]) for b in range(batch)]) if c["value_norm"] else None
    for b in range(batch):
        for g in range(kv):
            x = _scores64(q, k, b, g, group)
            if scores is not None:
                scores[b, g * group:(g + 1) * group] = x
            u = _pool64(x[:, : n - win], c["pool"], c["kernel"])
            if rho is not None:
                u = u * rho[b, g, : n - win]
            utility[b, g] = (u * wh[g * group:(g + 1) * group, None]).amax(0)
    out = {"utility": utility, "tau": None, "budget": None, "idx": None, "count": None, "k_out": None, "v_out": None}
    if scores is not None:
        out["scores"] = scores
    if rho is not None:
        out["rho"] = rho
    return out
