"""Timed cases of the eviction + decode path, through the package's public calls.

Each case is one piece of work a program that serves requests has this library
do: a prompt's prefill attention, its scores, the selection and compaction that
evict a fraction of its KV cache, the whole eviction, and decode steps over the
caches that remain.  `listed` names the sizes reported, `draw` gives others of
the same ranges, `prepare` makes what the program holds before the call,
`run` is the call, `work` what it cannot do without, and `exact` the same
result in float64 by plain torch.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2512_21859_amd import _lib
from paper_2512_21859_amd.pipeline import Evictor, run_decode

DT = {"bf16": torch.bfloat16, "fp32": torch.float32}
ESZ = {"bf16": 2, "fp32": 4}
PAGE = _lib.V_TILE


def listed():
    qwen = dict(Hq=28, Hkv=4, d=128, dtype="bf16")       # the 28-layer model shape
    long = dict(Hq=32, Hkv=8, d=128, dtype="bf16")       # the long-context shape
    return [
        # an eight-token reply over one layer of an 8k prompt, half evicted: the
        # smallest decode calls, replayed from a graph as a server does
        dict(name="decode_8k", kind="decode", how="graph", layers=1, B=1, lo=8192, hi=8192,
             alpha=0.5, steps=8, **qwen),
        # one token of the whole 28-layer stack at the 32k context, half
        # evicted: every layer's cache streams from HBM
        dict(name="decode_stack_32k", kind="decode", how="graph", layers=28, B=1, lo=32768,
             hi=32768, alpha=0.5, steps=1, **qwen),
        # decode calls over a 131k prompt's cache, half evicted
        dict(name="decode_131k", kind="decode", how="calls", layers=1, B=1, lo=131072, hi=131072,
             alpha=0.5, steps=2, **long),
        # steps of a running batch of 16 requests with ragged lengths and
        # ratios over paged caches
        dict(name="decode_paged_16", kind="decode", how="paged", layers=1, B=16, lo=1024, hi=16384,
             alpha=-1.0, steps=4, **qwen),
        # a short fp32 request: the smallest calls of all, made one by one
        dict(name="decode_fp32_512", kind="decode", how="calls", layers=1, B=1, lo=512, hi=512,
             alpha=0.5, steps=4, Hq=2, Hkv=1, d=64, dtype="fp32"),
        # the whole eviction of one layer of an 8k prompt
        dict(name="evict_8k", kind="evict", scorer="snapkv", B=1, lo=8192, hi=8192, w=32, pool=7,
             alpha=0.5, **qwen),
        # window scores of an admission batch of eight ragged prompts
        dict(name="score_ragged_8", kind="score", scorer="snapkv", B=8, lo=1024, hi=16384, w=32,
             pool=7, **qwen),
        # window scores of one layer of a 131k prompt
        dict(name="score_131k", kind="score", scorer="snapkv", B=1, lo=131072, hi=131072, w=64,
             pool=7, **long),
        # accumulated-attention scores (every prompt query) of a 4k prompt
        dict(name="h2o_4k", kind="score", scorer="h2o", B=1, lo=4096, hi=4096, w=32, pool=1, **qwen),
        # selection and compaction of one layer of a 32k prompt
        dict(name="keep_32k", kind="keep", B=1, lo=32768, hi=32768, w=32, pool=7, alpha=0.5, **qwen),
        # prefill attention of a short prompt of odd length
        dict(name="prefill_1k", kind="prefill", B=1, lo=1001, hi=1001, w=32, **qwen),
        # prefill attention of a long prompt, with the window's statistics
        dict(name="prefill_16k", kind="prefill", B=1, lo=16384, hi=16384, w=32, **qwen),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "evict", "score", "score", "keep", "prefill", "prefill"])
    Hq, Hkv, d = rng.choice([(28, 4, 128), (28, 4, 128), (32, 8, 128), (16, 2, 128), (8, 8, 128),
                             (12, 4, 64), (14, 2, 64)])
    c = dict(kind=kind, Hq=Hq, Hkv=Hkv, d=d,
             dtype="fp32" if kind != "prefill" and rng.random() < 0.2 else "bf16")
    alpha = round(rng.uniform(0.05, 0.95), 3)
    if kind == "decode":
        how = rng.choice(["graph", "calls", "paged"])
        B = rng.randint(2, 16) if how == "paged" or rng.random() < 0.2 else 1
        hi = _log(rng, 200, 131072 // B)
        lo = max(100, hi // 8) if B > 1 else hi
        layers = rng.choice([1, 4, 12]) if how == "graph" and B == 1 else 1
        c.update(how=how, layers=layers, B=B, lo=lo, hi=hi, alpha=-1.0 if B > 1 else alpha,
                 steps=rng.choice([1, 2, 4]))
        return c
    w = rng.choice([16, 32, 32, 64])
    if kind == "prefill":
        B = rng.choice([1, 1, 2, 4])
        hi = _log(rng, 100, 16384 // B)
        c.update(B=B, lo=max(64, hi // 4) if B > 1 else hi, hi=hi, w=w)
        return c
    c.update(w=w, pool=rng.choice([1, 5, 7]))
    if kind == "score":
        scorer = rng.choice(["snapkv", "snapkv", "snapkv_avg", "knorm", "h2o"])
        B = rng.choice([1, 1, 1, 3, 8])
        top = (131072 if Hkv == 8 else 65536) if scorer != "h2o" else 4096
        hi = _log(rng, 600, top // B) if scorer != "h2o" else _log(rng, 300, 4096 // min(B, 3))
        B = min(B, 3) if scorer == "h2o" else B
        c.update(scorer=scorer, B=B, lo=max(150, hi // 8) if B > 1 else hi, hi=hi)
        return c
    B = rng.choice([1, 1, 2, 6])
    hi = _log(rng, 400, (65536 if kind == "keep" else 12000) // B)
    c.update(B=B, lo=max(150, hi // 8) if B > 1 else hi, hi=hi, alpha=-1.0 if B > 1 else alpha)
    if kind == "evict":
        c["scorer"] = rng.choice(["snapkv", "snapkv", "snapkv_avg", "knorm"])
    return c


def lengths(c):
    """Prompt length of each sequence: `hi` for one, and the others spread over lo..hi."""
    r = random.Random(c["B"] * 1000003 + c["lo"] * 31 + c["hi"])
    return [c["hi"]] + [r.randint(c["lo"], c["hi"]) for _ in range(c["B"] - 1)]


def ratios(c):
    """Eviction ratio of each sequence (alpha < 0: spread over [0, 0.9))."""
    r = random.Random(c["B"] * 7919 + c["hi"])
    return [c["alpha"] if c["alpha"] >= 0 else r.uniform(0.0, 0.9) for _ in range(c["B"])]


def kept(c):
    w = c.get("w", 32)
    return [_lib.tb_keep_count(n, a, w) for n, a in zip(lengths(c), ratios(c))]


def _gen(seed, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    return g


def _randn(g, shape, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)


def _prompt(c, g, every_query=False):
    """Queries and K / V of the prompts: normal keys, 2% of them pulled towards
    one direction per KV head (the skew that attention has in earnest)."""
    dt, L = DT[c["dtype"]], lengths(c)
    B, Hq, Hkv, d, Lmax = c["B"], c["Hq"], c["Hkv"], c["d"], max(L)
    q = _randn(g, (B, Hq, Lmax if every_query else c["w"], d), dt)
    k = torch.randn((B, Hkv, Lmax, d), generator=g, device="cuda")
    u = torch.randn((B, Hkv, 1, d), generator=g, device="cuda")
    heavy = torch.rand((B, Hkv, Lmax, 1), generator=g, device="cuda") < 0.02
    k += heavy * (2.0 * math.sqrt(d) * u / u.norm(dim=-1, keepdim=True))
    for b, n in enumerate(L):
        k[b, :, n:] = 0
    v = _randn(g, (B, Hkv, Lmax, d), dt)
    return q, k.to(dt), v


def prepare(c, seed):
    g = _gen(seed)
    return {"decode": _prepare_decode, "evict": _prepare_evict, "score": _prepare_evict,
            "keep": _prepare_keep, "prefill": _prepare_prefill}[c["kind"]](c, g)


def run(s):
    return _RUN[s["kind"]](s)


# ------------------------------------------------------------------- decode
def _prepare_decode(c, g):
    """Caches as an eviction left them (kept rows, then room for the reply) and
    the tokens' q / k / v; paged ones with their pages scattered."""
    dt, n = DT[c["dtype"]], kept(c)
    nl, B, Hq, Hkv, d, T = c["layers"], c["B"], c["Hq"], c["Hkv"], c["d"], c["steps"]
    NB = nl * B
    s = dict(kind="decode", how=c["how"], T=T, layers=nl, B=B,
             q=_randn(g, (T, NB, Hq, d), dt), kn=_randn(g, (T, NB, Hkv, d), dt),
             vn=_randn(g, (T, NB, Hkv, d), dt), out=torch.zeros((T, NB, Hq, d), dtype=dt, device="cuda"),
             len0=torch.tensor(n * nl, dtype=torch.int32, device="cuda"), n=n)
    if c["how"] == "paged":
        need = [-(-(m + T) // PAGE) for m in n]
        order = torch.randperm(sum(need), generator=_gen(seed=sum(need), dev="cpu")).tolist()
        table = torch.zeros((B, max(need)), dtype=torch.int32)
        for b in range(B):
            mine = [order.pop() for _ in range(need[b])]
            table[b] = torch.tensor(mine + [mine[-1]] * (max(need) - len(mine)), dtype=torch.int32)
        s["table"], s["kv_len"] = table.cuda(), s["len0"].clone()
        s["k"] = _randn(g, (sum(need), Hkv, PAGE, d), dt)
        s["v"] = _randn(g, (sum(need), Hkv, PAGE, d), dt)
        nb = _lib.tb_workspace_bytes(_lib.TB_OP_DECODE, B, 0, Hq, Hkv, d, 0, max(need) * PAGE)
        s["ws"] = torch.zeros((max(nb, 1),), dtype=torch.uint8, device="cuda")
        return s
    if nl == 1:
        cache = _lib.KVCache(B, Hq, Hkv, max(n) + T, d, dt)
        cache.k.copy_(_randn(g, cache.k.shape, dt))
        cache.v.copy_(_randn(g, cache.v.shape, dt))
        for b, m in enumerate(n):
            cache.k[b, :, m:] = 0
            cache.v[b, :, m:] = 0
        cache.kv_len.copy_(s["len0"])
        s["cache"], s["k"], s["v"], s["kv_len"], s["ws"] = cache, cache.k, cache.v, cache.kv_len, cache.ws
    else:
        # the layers' caches stacked on the batch axis, as a stacked eviction fills them
        one = _lib.KVCache(B, Hq, Hkv, max(n) + T, d, dt)
        s["ws"] = one.ws
        s["k"] = torch.zeros((NB,) + tuple(one.k.shape[1:]), dtype=dt, device="cuda")
        s["v"] = torch.zeros_like(s["k"])
        for i in range(NB):
            s["k"][i, :, :n[i % B]] = _randn(g, (Hkv, n[i % B], d), dt)
            s["v"][i, :, :n[i % B]] = _randn(g, (Hkv, n[i % B], d), dt)
        s["kv_len"] = s["len0"].clone()
    if c["how"] == "graph":
        graph, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(graph, stream=st):
            for t in range(T):
                for l in range(nl):
                    r = slice(l * B, (l + 1) * B)
                    _lib.tb_decode_attn(s["q"][t, r], s["kn"][t, r], s["vn"][t, r], s["k"][r], s["v"][r],
                                        s["kv_len"][r], s["out"][t, r], s["ws"], stream=st)
        torch.cuda.current_stream().wait_stream(st)
        s["graph"] = graph
    return s


def _run_decode(s):
    """A reply of T tokens from the prompt's cache: the lengths go back to the
    prompt's (as where several replies are sampled from one prompt), then T
    steps append a row and attend."""
    s["kv_len"].copy_(s["len0"])
    if s["how"] == "graph":
        s["graph"].replay()
    elif s["how"] == "paged":
        for t in range(s["T"]):
            _lib.tb_decode_attn_paged(s["q"][t], s["kn"][t], s["vn"][t], s["k"], s["v"], s["table"],
                                      s["kv_len"], s["out"][t], s["ws"])
    else:
        s["cache"].host_len = list(s["n"])
        run_decode(s["cache"], s["q"], s["kn"], s["vn"], s["out"])
    return {"out": s["out"], "len": s["kv_len"], "k": s["k"], "v": s["v"]}


def _exact_decode(c, seed):
    s = _prepare_decode(dict(c, how="paged" if c["how"] == "paged" else "calls"), _gen(seed)) \
        if c["layers"] == 1 else _prepare_decode(dict(c, how="rows"), _gen(seed))
    n, T, NB, G, d = s["n"], s["T"], s["layers"] * s["B"], c["Hq"] // c["Hkv"], c["d"]
    out = torch.empty(s["out"].shape, dtype=torch.float64, device="cuda")
    for i in range(NB):
        m = n[i % s["B"]]
        if c["how"] == "paged":
            pages = s["table"][i].long()
            rows = lambda x: x[pages].permute(1, 0, 2, 3).reshape(c["Hkv"], -1, d)[:, :m]  # noqa: E731
        else:
            rows = lambda x: x[i, :, :m]  # noqa: E731
        k = torch.cat([rows(s["k"]).double(), s["kn"][:, i].double().permute(1, 0, 2)], dim=1)
        v = torch.cat([rows(s["v"]).double(), s["vn"][:, i].double().permute(1, 0, 2)], dim=1)
        for t in range(T):
            for h in range(c["Hkv"]):
                q = s["q"][t, i, h * G:(h + 1) * G].double()
                p = torch.softmax(q @ k[h, :m + t + 1].T / math.sqrt(d), dim=-1)
                out[t, i, h * G:(h + 1) * G] = p @ v[h, :m + t + 1]
    return {"out": out, "len": None, "k": None, "v": None}


# -------------------------------------------------------- scores, eviction
def _prepare_evict(c, g):
    L = lengths(c)
    q, k, v = _prompt(c, g, every_query=c["scorer"] == "h2o")
    ev = Evictor(c["B"], max(L), c["Hq"], c["Hkv"], c["d"], c["w"], c["pool"], scorer=c["scorer"])
    ev.scores.zero_()
    ev.keep_idx.zero_()
    s = dict(kind=c["kind"], ev=ev, q=q, k=k, L=L)
    if c["kind"] == "evict":
        s["v"], s["alphas"] = v, ratios(c)
        s["cache"] = _lib.KVCache(c["B"], c["Hq"], c["Hkv"], max(kept(c)) + 32, c["d"], DT[c["dtype"]])
        s["cache"].k.zero_()
        s["cache"].v.zero_()
    return s


def _run_score(s):
    s["ev"].score(s["q"], s["k"], s["L"])
    return s["ev"].scores


def _run_evict(s):
    n = s["ev"].evict(s["q"], s["k"], s["v"], s["L"], s["alphas"], s["cache"])
    cache = s["cache"]
    return {"scores": s["ev"].scores, "keep": s["ev"].keep_idx, "n": n, "k": cache.k, "v": cache.v,
            "len": cache.kv_len}


def _exact_scores(c, seed):
    L, G, w, scorer = lengths(c), c["Hq"] // c["Hkv"], c["w"], c["scorer"]
    q, k, _ = _prompt(c, _gen(seed), every_query=scorer == "h2o")
    out = torch.zeros((c["B"], c["Hkv"], max(L)), dtype=torch.float64, device="cuda")
    for b, n in enumerate(L):
        for h in range(c["Hkv"]):
            kk = k[b, h, :n].double()
            if scorer == "knorm":
                out[b, h, :n - w] = -kk[:n - w].norm(dim=-1)
                continue
            rows = n if scorer == "h2o" else w
            at = torch.arange(n - rows, n, device="cuda")
            a = torch.zeros(n, dtype=torch.float64, device="cuda")
            for i in range(h * G, (h + 1) * G):
                s = q[b, i, :rows].double() @ kk.T / math.sqrt(c["d"])
                s.masked_fill_(torch.arange(n, device="cuda")[None, :] > at[:, None], -math.inf)
                a += torch.softmax(s, dim=-1).sum(dim=0)
            if scorer == "h2o":
                out[b, h, :n] = a
                continue
            a, p = a[None, None, :n - w], c["pool"]
            if scorer == "snapkv":
                a = torch.nn.functional.max_pool1d(a, p, 1, p // 2)
            else:
                a = torch.nn.functional.avg_pool1d(a, p, 1, p // 2, count_include_pad=True)
            out[b, h, :n - w] = a[0, 0]
    return out


# ----------------------------------------------- selection and compaction
def _prepare_keep(c, g):
    """Scores as the window scorer leaves them: positive, skewed, with the
    plateaus that max-pooling makes."""
    L = lengths(c)
    _, k, v = _prompt(c, g)
    ev = Evictor(c["B"], max(L), c["Hq"], c["Hkv"], c["d"], c["w"], c["pool"])
    raw = torch.exp(0.5 * torch.randn(ev.scores.shape, generator=g, device="cuda")) / max(L)
    ev.scores.copy_(torch.nn.functional.max_pool1d(raw, c["pool"], 1, c["pool"] // 2))
    ev.keep_idx.zero_()
    cache = _lib.KVCache(c["B"], c["Hq"], c["Hkv"], max(kept(c)) + 32, c["d"], DT[c["dtype"]])
    cache.k.zero_()
    cache.v.zero_()
    return dict(kind="keep", ev=ev, k=k, v=v, L=L, alphas=ratios(c), cache=cache)


def _run_keep(s):
    cache = s["cache"]
    n = s["ev"].select(s["L"], s["alphas"])
    cache.compact_from(s["k"], s["v"], s["ev"].keep_idx, n)
    return {"keep": s["ev"].keep_idx, "n": n, "k": cache.k, "v": cache.v, "len": cache.kv_len}


# ------------------------------------------------------------------ prefill
def _prepare_prefill(c, g):
    L = lengths(c)
    q, k, v = _prompt(c, g, every_query=True)
    stats = torch.zeros((c["B"], c["Hq"], c["w"], 2), dtype=torch.float32, device="cuda")
    return dict(kind="prefill", q=q, k=k, v=v, L=L, w=c["w"], out=torch.zeros_like(q), stats=stats)


def _run_prefill(s):
    _lib.tb_prefill_attn(s["q"], s["k"], s["v"], s["L"], s["out"], s["w"], s["stats"])
    return {"out": s["out"], "stats": s["stats"]}


def _exact_prefill(c, seed):
    L, G, w, d = lengths(c), c["Hq"] // c["Hkv"], c["w"], c["d"]
    q, k, v = _prompt(c, _gen(seed), every_query=True)
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    stats = torch.zeros((c["B"], c["Hq"], w, 2), dtype=torch.float64, device="cuda")
    for b, n in enumerate(L):
        for h in range(c["Hq"]):
            kk, vv = k[b, h // G, :n].double(), v[b, h // G, :n].double()
            for r in range(0, n, 4096):
                e = min(r + 4096, n)
                s = q[b, h, r:e].double() @ kk[:e].T / math.sqrt(d)
                at = torch.arange(r, e, device="cuda")
                s.masked_fill_(torch.arange(e, device="cuda")[None, :] > at[:, None], -math.inf)
                m = s.max(dim=-1, keepdim=True).values
                p = torch.exp(s - m)
                z = p.sum(dim=-1, keepdim=True)
                out[b, h, r:e] = (p @ vv[:e]) / z
                x = max(r, n - w)
                if x < e:
                    stats[b, h, x - (n - w):e - (n - w), 0] = m[x - r:, 0]
                    stats[b, h, x - (n - w):e - (n - w), 1] = z[x - r:, 0]
    return {"out": out, "stats": stats}


_RUN = {"decode": _run_decode, "evict": _run_evict, "score": _run_score, "keep": _run_keep,
        "prefill": _run_prefill}


def work(c):
    """Bytes (inputs read once, outputs written once) and operations of one pass."""
    L, e, Hq, Hkv, d = lengths(c), ESZ[c["dtype"]], c["Hq"], c["Hkv"], c["d"]
    if c["kind"] == "decode":
        rows = c["layers"] * sum(m + t + 1 for m in kept(c) for t in range(c["steps"]))
        tokens = c["layers"] * c["B"] * c["steps"]
        return {"bytes": e * d * (2 * Hkv * rows + tokens * (2 * Hq + 2 * Hkv)), "flops": 4 * Hq * d * rows}
    if c["kind"] == "prefill":
        return {"bytes": e * d * sum(L) * (2 * Hq + 2 * Hkv),
                "flops": sum(2 * Hq * d * n * (n + 1) for n in L)}
    score = {"bytes": 0, "flops": 0}
    if c["kind"] != "keep":
        queries = {"knorm": 0, "h2o": sum(L)}.get(c["scorer"], c["B"] * c["w"])
        score["bytes"] = Hkv * sum(L) * (e * d + 4) + e * d * Hq * queries
        score["flops"] = {"knorm": 2 * Hkv * d * sum(L), "h2o": sum(Hq * d * n * (n + 1) for n in L)}.get(
            c["scorer"], 2 * Hq * c["w"] * d * sum(L))
    if c["kind"] == "score":
        return score
    keep = Hkv * (4 * sum(L) + sum(kept(c)) * (4 + 4 * e * d))
    return {"bytes": score["bytes"] + keep, "flops": score["flops"]}


def tolerance(c):
    """About four times the error that the path shows against `exact`."""
    if c["kind"] == "keep":
        return "exact"
    if c["kind"] == "prefill":
        return {"rel": 9e-3, "max": 0.1}
    if c["kind"] == "decode":
        return {"rel": 9e-3, "max": 0.1} if c["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}
    # scores are float64 sums rounded to fp32; two correct sums may round
    # apart, and the kept positions follow the scores
    return {"rel": 2e-7, "max": 1e-6, "differ": 1e-2}


def exact(c, seed):
    if c["kind"] == "decode":
        return _exact_decode(c, seed)
    if c["kind"] == "prefill":
        return _exact_prefill(c, seed)
    if c["kind"] == "score":
        return _exact_scores(c, seed)
    if c["kind"] == "evict":
        return {"scores": _exact_scores(c, seed), "keep": None, "n": None, "k": None, "v": None, "len": None}
    return None
