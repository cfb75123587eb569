"""Performance cases of the verifier path: what a serving stack has it do.

A case names one entry point (or the short chain of entry points that a
program calls together) and its sizes:

- ``decide``:    token_features -> request_aggregate -> route on a batch of
                 finished requests (offline scoring, the summary verifier);
- ``verdict``:   feature_sequence -> verifier_head -> route, from the logits
                 of finished requests to the decision of the paper's verifier;
- ``head``:      verifier_head alone, on input sequences already collected;
- ``stream``:    a stretch of decode steps over request slots, then their
                 verdicts (StreamState.step / .finish);
- ``sample``:    one decode step that draws the tokens and verifies them;
- ``calibrate``: the threshold of a validation pool.

Logits follow the repository's row model (z = s g + a spike), made from the
seed alone; ids are drawn from softmax(z / T), inside the nucleus with top-p.
"""

import math

import numpy as np
import torch

import paper_2608_28726_amd as pr
from paper_2608_28726_amd import workloads as wl

DEV = "cuda"
Q = 0.1        # quantile of the request summaries
TAU = 0.5      # ship threshold
TOP_K = 20     # K of the top-K entropy
CHUNK = 256 * 262144  # logits handled together while inputs or exact values are made


def listed():
    return [
        # The reference batch: 8 requests of 64 tokens, V = 32,000 float32. Latency and launches count.
        dict(name="decide_8x64_v32000_f32", op="decide", n_req=8, len_lo=64, len_hi=64, V=32000, dtype="f32", T=1.0,
             P=0.0),
        # The benchmark's batch: 64 ragged requests, V = 151,936 bfloat16, T = 0.7. The largest read.
        dict(name="decide_64req_v151936_bf16", op="decide", n_req=64, len_lo=16, len_hi=512, V=151936, dtype="bf16",
             T=0.7, P=0.0),
        # A vocabulary that is no multiple of a vector: every row starts and ends unaligned.
        dict(name="decide_20req_v50257_bf16", op="decide", n_req=20, len_lo=1, len_hi=80, V=50257, dtype="bf16",
             T=1.0, P=0.0),
        # Top-p on a float32 vocabulary of 262,144: decoding configurations with nucleus sampling.
        dict(name="decide_topp_32x128_v262144_f32", op="decide", n_req=32, len_lo=128, len_hi=128, V=262144,
             dtype="f32", T=0.7, P=0.9),
        # One request has ended and its verdict is wanted: the routing signal's latency.
        dict(name="verdict_1req_v151936_bf16", op="verdict", n_req=1, len_lo=93, len_hi=93, V=151936, dtype="bf16",
             T=0.7, P=0.0),
        # A batch of finished requests decoded with top-p, to the paper's verifier and its decision.
        dict(name="verdict_topp_16req_v151936_bf16", op="verdict", n_req=16, len_lo=16, len_hi=512, V=151936,
             dtype="bf16", T=0.7, P=0.9),
        # The transformer head on the sequences of 64 finished requests.
        dict(name="head_64req", op="head", n_req=64, len_lo=16, len_hi=512),
        # Eight decode steps of 256 concurrent requests and their verdicts.
        dict(name="stream_256slots_v151936_bf16", op="stream", n_req=256, steps=8, max_len=1024, V=151936,
             dtype="bf16", T=1.0, P=0.0),
        # A small decode batch sampled with top-p: eight steps of 16 slots.
        dict(name="stream_topp_16slots_v151936_bf16", op="stream", n_req=16, steps=8, max_len=1024, V=151936,
             dtype="bf16", T=0.7, P=0.9),
        # One decode step of 32 requests that draws the tokens and verifies them in one pass.
        dict(name="sample_32rows_v151936_bf16", op="sample", n_req=32, V=151936, dtype="bf16", T=0.7, seq=0),
        # Thresholds of an ordinary validation pool and of a large one.
        dict(name="calibrate_8192", op="calibrate", n=8192, fraction=0.6),
        dict(name="calibrate_1048576", op="calibrate", n=1048576, fraction=0.6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("decide", "decide", "verdict", "verdict", "head", "stream", "stream", "sample", "calibrate"))
    if op == "calibrate":
        return dict(op=op, n=_log_int(rng, 1000, 1 << 20), fraction=round(rng.uniform(0.05, 0.95), 3))
    if op == "head":
        lo = _log_int(rng, 1, 64)
        return dict(op=op, n_req=_log_int(rng, 1, 64), len_lo=lo, len_hi=_log_int(rng, lo, 512))
    dtype = rng.choice(("bf16", "bf16", "f32"))
    V = rng.choice((32000, 50257, 65536, 128003, 131072, 151936, 151936, 262144))
    c = dict(op=op, V=V, dtype=dtype, T=rng.choice((0.3, 0.5, 0.7, 1.0, 1.2)))
    P = rng.choice((0.0, 0.0, 0.8, 0.9, 0.95))
    # bytes and, with top-p, logits stay below those of the largest listed cases
    most = (4.0e9 if P == 0.0 else 1.6e9) / (V * (2 if dtype == "bf16" else 4))
    if op == "stream":
        n = _log_int(rng, 1, 256)
        c.update(n_req=n, steps=max(1, min(rng.randint(4, 12), int(most / n))), P=P, max_len=rng.choice((0, 1024)))
    elif op == "sample":
        c.update(n_req=_log_int(rng, 1, min(8192, int(most))), seq=rng.randint(0, 1))
    else:
        rows = _log_int(rng, 4, most)
        lo = _log_int(rng, 1, 128)
        hi = max(lo, min(_log_int(rng, lo, 512), rows))
        c.update(n_req=max(1, min(512, rows // hi)), len_lo=min(lo, hi), len_hi=hi, P=P)
    return c


# ---------------------------------------------------------------------------
# Sizes

def _lengths(case):
    """Request lengths: part of the case, the same for every seed."""
    rng = np.random.default_rng([case["n_req"], case["len_lo"], case["len_hi"]])
    return rng.integers(case["len_lo"], case["len_hi"] + 1, size=case["n_req"]).astype(np.int64)


def _offsets(case):
    off = np.zeros(case["n_req"] + 1, dtype=np.int32)
    off[1:] = np.cumsum(_lengths(case))
    return off


def _n_rows(case):
    if case["op"] in ("stream", "sample"):
        return case["n_req"]
    return int(_lengths(case).sum())


def _head_flops(lengths):
    """Multiply-adds as two: projections and feed-forward per token, scores and values per pair of tokens."""
    n, pairs = float(lengths.sum()), float((lengths.astype(np.float64) ** 2).sum())
    per_layer = n * 2 * (64 * 192 + 64 * 64 + 2 * 64 * 128) + pairs * 2 * 2 * 64
    return n * 2 * 4 * 64 + 2 * per_layer


def work(case):
    op = case["op"]
    if op == "calibrate":
        return {"bytes": 4 * case["n"] + 8, "flops": 0}
    if op == "head":
        L = _lengths(case)
        return {"bytes": int(L.sum()) * 16 + 4 * (case["n_req"] + 1) + 4 * 67329 + 4 * case["n_req"],
                "flops": _head_flops(L)}
    n, V = _n_rows(case), case["V"]
    item = 2 if case["dtype"] == "bf16" else 4
    row = V * item + 8 + (4 if case.get("P") else 0)
    flops = 6.0 * n * V  # scale, exp, sum and entropy sum per logit
    if op == "stream":
        return {"bytes": case["steps"] * n * (row + 4) + n * 57, "flops": flops * case["steps"]}
    if op == "sample":
        return {"bytes": n * (V * item + 4 + 4 + 40 + (16 if case["seq"] else 0)), "flops": flops}
    if op == "decide":
        return {"bytes": n * (row + 40) + case["n_req"] * 61, "flops": flops}
    return {"bytes": n * (row + 16) + case["n_req"] * 9 + 4 * 67329, "flops": flops + _head_flops(_lengths(case))}


# ---------------------------------------------------------------------------
# Inputs

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 1)
    return g


def _make_logits(n, V, dtype, T, P, g, want_ids=True):
    """Logits [n, V] of the row model and one drawn id per row."""
    out = torch.empty(n, V, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV)
    ids = torch.empty(n, dtype=torch.int32, device=DEV)
    s = torch.empty(n, 1, device=DEV).uniform_(1.0, 4.0, generator=g)
    h = torch.empty(n, 1, device=DEV).uniform_(0.0, 15.0, generator=g)
    j = torch.randint(0, V, (n, 1), generator=g, device=DEV)
    step = max(1, CHUNK // V)
    for a in range(0, n, step):
        b = min(n, a + step)
        z = torch.empty(b - a, V, device=DEV).normal_(generator=g).mul_(s[a:b])
        z.scatter_add_(1, j[a:b], h[a:b])
        out[a:b] = z
        if not want_ids:
            continue
        z = out[a:b].float()
        p = torch.softmax(z / T, dim=1)
        race = torch.empty_like(p).exponential_(generator=g)
        y = torch.argmax(p / race.clamp_(min=1e-30), dim=1, keepdim=True)
        if P:  # outside the nucleus: the most likely token instead
            above = (p * (z > z.gather(1, y))).sum(1, keepdim=True)
            y = torch.where(above < 0.999 * P, y, torch.argmax(z, dim=1, keepdim=True))
        ids[a:b] = y.squeeze(1).to(torch.int32)
    return out, ids


def _make_X(lengths, g):
    """Input sequences of the head as decoding gives them: log-prob, max-prob, -entropy, position."""
    n = int(lengths.sum())
    u = torch.rand(n, 3, generator=g, device=DEV)
    m = u[:, 0].sqrt().clamp(0.02, 0.9999)
    X = torch.empty(n, 4, device=DEV)
    X[:, 0] = torch.where(u[:, 1] < m, m.log(), ((1 - m) * (0.02 + 0.9 * u[:, 2])).log())
    X[:, 1] = m
    X[:, 2] = -(1 - m) * 2.5 + m * m.log()
    pos = np.concatenate([np.arange(1, k + 1, dtype=np.float64) / k for k in lengths])
    X[:, 3] = torch.from_numpy(pos.astype(np.float32)).to(DEV)
    return X


def _head_weights():
    return torch.from_numpy(wl.head_weights()).to(DEV)


def prepare(case, seed):
    g = _generator(seed)
    op = case["op"]
    st = {"case": case}
    if op == "calibrate":
        u = torch.rand(case["n"], 7, generator=g, device=DEV, dtype=torch.float32)
        st["scores"] = torch.sort(u[:, :6], dim=1).values[:, 4].contiguous()  # Beta(5, 2): mostly confident
        st["scores"][u[:, 6] < 0.005] = float("nan")  # requests without a score
        return st
    if op == "head":
        L = _lengths(case)
        st["X"] = _make_X(L, g)
        st["offsets"] = torch.from_numpy(_offsets(case)).to(DEV)
        st["weights"] = _head_weights()
        st["max_len"] = int(L.max())
        return st
    n, T, P = _n_rows(case), case["T"], case.get("P", 0.0)
    st["T"] = torch.full((n,), T, device=DEV)
    st["P"] = torch.full((n,), P, device=DEV) if P else None
    if op == "stream":
        st["steps"] = [_make_logits(n, case["V"], case["dtype"], T, P, g) for _ in range(case["steps"])]
        st["slots"] = torch.randperm(n, generator=g, device=DEV).to(torch.int32)
        st["state"] = pr.StreamState(n, case["max_len"], q=Q)
        return st
    if op == "sample":
        st["logits"], _ = _make_logits(n, case["V"], case["dtype"], T, P, g, want_ids=False)
        st["seed"] = int(seed)
        st["offsets"] = torch.arange(n + 1, dtype=torch.int32, device=DEV) if case["seq"] else None
        return st
    st["logits"], st["ids"] = _make_logits(n, case["V"], case["dtype"], T, P, g)
    st["offsets"] = torch.from_numpy(_offsets(case)).to(DEV)
    if op == "verdict":
        st["weights"] = _head_weights()
        st["max_len"] = int(_lengths(case).max())
    return st


# ---------------------------------------------------------------------------
# One pass

def run(st):
    case = st["case"]
    op = case["op"]
    if op == "decide":
        f = pr.token_features(st["logits"], st["ids"], st["T"], top_p=st["P"])
        agg = pr.request_aggregate(f, st["offsets"], q=Q)
        ship, n_ship = pr.route(agg["score"], TAU)
        return {"features": f, "agg": agg, "ship": ship, "n_ship": n_ship}
    if op == "verdict":
        X = pr.feature_sequence(st["logits"], st["ids"], st["T"], st["offsets"], top_p=st["P"], top_k=TOP_K)
        score = pr.verifier_head(X, st["offsets"], st["weights"], max_len=st["max_len"])
        ship, n_ship = pr.route(score, TAU)
        return {"X": X, "score": score, "ship": ship, "n_ship": n_ship}
    if op == "head":
        return {"score": pr.verifier_head(st["X"], st["offsets"], st["weights"], max_len=st["max_len"])}
    if op == "stream":
        state = st["state"]
        for logits, ids in st["steps"]:
            state.step(logits, st["slots"], ids, st["T"], top_p=st["P"])
        return state.finish(st["slots"], TAU)
    if op == "sample":
        ids, f, X = pr.sample_features(st["logits"], st["T"], st["seed"], offsets=st["offsets"], top_k=TOP_K)
        return {"ids": ids, "features": f, "X": X} if X is not None else {"ids": ids, "features": f}
    tau, n_ship = pr.calibrate_threshold(st["scores"], case["fraction"])
    return {"tau": tau, "n_ship": n_ship}


def tolerance(case):
    op = case["op"]
    if op == "calibrate":
        return "exact"  # tau is one of the scores
    if op == "head":
        return {"rel": 4e-6, "max": 2e-5}
    # 32-bit sums of exponentials over the vocabulary
    return {"rel": 1e-5, "max": 2e-4}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits

def _exact_rows(logits, ids, T, P, top_k):
    """Per-row features, and the top-K entropy, of every row (float64; ids None: no sampled token)."""
    n, V = logits.shape
    names = ("max_logit", "lse", "entropy", "logprob", "maxprob", "margin", "rank", "argmax", "cutoff", "topk_entropy")
    out = {k: torch.empty(n, dtype=torch.float64, device=DEV) for k in names}
    col = torch.arange(V, device=DEV)
    T = float(np.float32(T))
    P = float(np.float32(P))
    step = max(1, CHUNK // 4 // V)
    for a in range(0, n, step):
        b = min(n, a + step)
        z = logits[a:b].double()
        M = z.max(1, keepdim=True).values
        out["argmax"][a:b] = torch.where(z == M, col, V).min(1).values
        top = torch.topk(z, max(top_k, 2), dim=1).values
        out["max_logit"][a:b] = M[:, 0] / T
        out["margin"][a:b] = (top[:, 0] - top[:, 1]) / T
        u = (z - M) / T
        e = torch.exp(u)
        if P:
            us = torch.sort(u, dim=1, descending=True).values
            es = torch.exp(us)
            cum = es.cumsum(1)
            k = (cum < P * cum[:, -1:]).sum(1, keepdim=True).clamp_(max=V - 1) + 1
            inside = col < k
            S = (es * inside).sum(1)
            E = (es * us * inside).sum(1)
            del us, es, cum, inside
        else:
            k = torch.full((b - a, 1), V, device=DEV)
            S = e.sum(1)
            E = (e * u).sum(1)
        lnS = S.log()
        out["lse"][a:b] = M[:, 0] / T + lnS
        out["entropy"][a:b] = lnS - E / S
        out["maxprob"][a:b] = 1.0 / S
        out["cutoff"][a:b] = k[:, 0].double()
        j = torch.arange(top.shape[1], device=DEV)
        ut = (top - M) / T
        p = torch.exp(ut) / S[:, None]
        out["topk_entropy"][a:b] = -torch.where(j < k.clamp(max=top_k), p * (ut - lnS[:, None]), 0.0).sum(1)
        if ids is not None:
            y = ids[a:b].long()[:, None]
            zy = z.gather(1, y)
            rank = ((z > zy) | ((z == zy) & (col < y))).sum(1) + 1
            out["rank"][a:b] = rank.double()
            lp = (zy[:, 0] - M[:, 0]) / T - lnS
            out["logprob"][a:b] = torch.where(rank <= k[:, 0], lp, -math.inf)
    return out


def _exact_summary(f, offsets):
    """Per-request summaries of (logprob, maxprob, -entropy, margin), score included."""
    cols = torch.stack([f["logprob"], f["maxprob"], -f["entropy"], f["margin"]], 1).cpu().numpy()
    R = len(offsets) - 1
    mean, mn, qu = (np.full((R, 4), np.nan) for _ in range(3))
    for i in range(R):
        x = cols[offsets[i]:offsets[i + 1]]
        if len(x):
            mean[i], mn[i] = x.mean(0), x.min(0)
            qu[i] = np.sort(x, axis=0)[max(1, math.ceil(Q * len(x))) - 1]
    to = lambda v: torch.from_numpy(v)  # noqa: E731
    return {"count": to(np.diff(offsets).astype(np.int32)), "mean": to(mean), "min": to(mn), "quant": to(qu),
            "score": to(mean[:, 1].copy())}


def _exact_ship(score):
    ship = (score >= TAU).to(torch.uint8)
    return ship, ship.sum().to(torch.int32).reshape(1)


def _exact_head(X, lengths):
    """The transformer head in float64 (seeded weights): one score per request."""
    w = torch.from_numpy(wl.head_weights()).to(DEV).double()
    at = 0

    def take(*shape):
        nonlocal at
        k = int(np.prod(shape))
        at += k
        return w[at - k:at].reshape(shape)

    def norm(h, g, b):
        mu = h.mean(1, keepdim=True)
        return (h - mu) / ((h - mu).square().mean(1, keepdim=True) + 1e-5).sqrt() * g + b

    n = X.shape[0]
    pos = torch.from_numpy(np.concatenate([np.arange(k, dtype=np.float64) for k in lengths])).to(DEV)
    angle = pos[:, None] * torch.exp(torch.arange(32, device=DEV).double() * (-2.0 / 64 * math.log(10000.0)))
    pe = torch.stack([angle.sin(), angle.cos()], 2).reshape(n, 64)
    h = X.double() @ take(64, 4).T + take(64) + pe
    ends = np.concatenate([[0], np.cumsum(lengths)])
    for _ in range(2):
        qkv = h @ take(192, 64).T + take(192)
        Wo, bo, g1, b1 = take(64, 64), take(64), take(64), take(64)
        W1, c1, W2, c2, g2, b2 = take(128, 64), take(128), take(64, 128), take(64), take(64), take(64)
        att = torch.empty(n, 64, dtype=torch.float64, device=DEV)
        for i in range(len(lengths)):
            x = qkv[ends[i]:ends[i + 1]]
            for hd in range(4):
                q, k, v = (x[:, 64 * m + 16 * hd:64 * m + 16 * hd + 16] for m in range(3))
                att[ends[i]:ends[i + 1], 16 * hd:16 * hd + 16] = torch.softmax(q @ k.T / 4.0, 1) @ v
        h = norm(h + att @ Wo.T + bo, g1, b1)
        h = norm(h + torch.relu(h @ W1.T + c1) @ W2.T + c2, g2, b2)
    wo, b = take(64), take(1)
    return torch.stack([1 / (1 + torch.exp(-(h[ends[i]:ends[i + 1]].mean(0) @ wo + b[0])))
                        for i in range(len(lengths))])


def _features(f, sampled=True):
    out = {k: f[k] for k in ("max_logit", "lse", "entropy", "maxprob", "margin")}
    out["logprob"] = f["logprob"] if sampled else None
    out["rank"] = f["rank"].to(torch.int32) if sampled else None
    out["argmax"] = f["argmax"].to(torch.int32)
    out["cutoff"] = f["cutoff"].to(torch.int32)
    out["flags"] = torch.zeros_like(out["argmax"])
    return out


def exact(case, seed):
    st = prepare(case, seed)
    op = case["op"]
    if op == "calibrate":
        s = st["scores"].double()
        s = torch.sort(s[~s.isnan()], descending=True).values
        k = max(1, math.ceil(case["fraction"] * s.numel()))
        return {"tau": s[k - 1].reshape(1), "n_ship": (s >= s[k - 1]).sum().to(torch.int32).reshape(1)}
    if op == "head":
        return {"score": _exact_head(st["X"], _lengths(case))}
    T, P = case["T"], case.get("P", 0.0)
    if op == "stream":
        n, steps = case["n_req"], case["steps"]
        rows = [_exact_rows(z, ids, T, P, TOP_K) for z, ids in st["steps"]]
        f = {k: torch.stack([r[k] for r in rows], 1).reshape(-1) for k in rows[0]}
        agg = _exact_summary(f, np.arange(n + 1, dtype=np.int64) * steps)
        if case["max_len"] == 0:
            agg["quant"] = None  # an estimate
        return {**agg, "ship": _exact_ship(agg["score"])[0]}
    if op == "sample":
        f = _exact_rows(st["logits"], None, T, 0.0, TOP_K)
        got = {"ids": None, "features": _features(f, sampled=False)}
        return {**got, "X": None} if case["seq"] else got
    f = _exact_rows(st["logits"], st["ids"], T, P, TOP_K)
    if op == "decide":
        agg = _exact_summary(f, _offsets(case))
        ship, n_ship = _exact_ship(agg["score"])
        return {"features": _features(f), "agg": agg, "ship": ship, "n_ship": n_ship}
    L = _lengths(case)
    pos = np.concatenate([np.arange(1, k + 1, dtype=np.float64) / k for k in L])
    X = torch.stack([f["logprob"], f["maxprob"], -f["topk_entropy"], torch.from_numpy(pos).to(DEV)], 1)
    score = _exact_head(X, L)
    ship, n_ship = _exact_ship(score)
    return {"X": X, "score": score, "ship": ship, "n_ship": n_ship}
