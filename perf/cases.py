"""The work that a program built on this library has it do, as cases to be timed.

Kinds of case (``case["kind"]``), each through the public binding:

* ``schedule``  the layers of one forward pass on a ledger: an anchor at layer
  0, then relay layers, with every layer's routes (what the attention backend
  takes), masks and counts, and the ledger's state at the end (kept for the
  next segment or saved);
* ``full``      full routing of one layer with the score of every route slot;
* ``pool``      chunk representations of one layer's token vectors;
* ``expand``    routed chunks to token ids, for backends that take token lists;
* ``attention`` sparse attention along given routes;
* ``prefill``   one layer from tokens to attention output: pooling of the
  query and key tokens, an anchor on the pooled chunks, sparse attention along
  its routes.

Sizes are those of the presets in ``paper_2609_07306_amd/synth.py`` and of the
benchmark's prefill point, cut to one anchor period or less.
"""
from __future__ import annotations

import math

import torch

from paper_2609_07306_amd import routerelay as rr

DEV = "cuda"


def _schedule(name, heads, kv, n, nk, d, dtype, k, m, r, causal, rho, layers, near_ties=False, sinks=0, recent=0,
              min_reuse=0, budgets=False):
    c = dict(kind="schedule", heads=heads, kv_heads=kv, n=n, nk=nk, d=d, dtype=dtype, k=k, m=m, r=r, causal=causal,
             rho=rho, layers=layers, near_ties=near_ties, sinks=sinks, recent=recent, min_reuse=min_reuse,
             budgets=budgets)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest calls: one head, a few launches of a tile or four each
        _schedule("tiny schedule", 1, 1, 128, 128, 64, "f32", 8, 4, 4, False, 0.3, 4),
        # the cross-layer drift workload: binary32 representations, two anchor
        # periods of a small model
        _schedule("drift schedule f32", 8, 8, 256, 256, 128, "f32", 16, 8, 8, False, 0.1, 8),
        # grouped-query causal prefill routing, one anchor period
        _schedule("gqa causal schedule", 32, 8, 512, 512, 128, "bf16", 32, 16, 16, True, 0.3, 8),
        # the scale workload the benchmark's headline is quoted on, one anchor
        # period; then at a drift where most rows keep their route
        _schedule("scale schedule", 32, 32, 1024, 1024, 128, "bf16", 32, 16, 16, False, 0.3, 8),
        _schedule("scale schedule low drift", 32, 32, 1024, 1024, 128, "bf16", 32, 16, 16, False, 0.01, 8),
        # long context: causal, duplicated keys, wide routes
        _schedule("long context schedule", 32, 32, 4096, 4096, 128, "bf16", 64, 32, 32, True, 0.6, 3, near_ties=True),
        # stateless routing of a layer, with the slots' scores
        dict(name="full routing", kind="full", heads=32, kv_heads=32, n=1024, nk=1024, d=128, dtype="bf16", k=32,
             causal=False, budgets=False),
        # odd sizes, more keys than queries, per-row route widths, binary32
        dict(name="full routing ragged f32", kind="full", heads=6, kv_heads=2, n=777, nk=1500, d=64, dtype="f32", k=24,
             causal=False, budgets=True),
        # one layer's query tokens of a long prefill
        dict(name="pool prefill", kind="pool", heads=32, tokens=65536, d=128, chunk=256, dtype="bf16"),
        # token lists of a causal layer's routes
        dict(name="expand tokens", kind="expand", heads=32, tokens=32768, chunk=64, k=32, causal=True),
        # attention of a causal grouped-query prefill along its routes
        dict(name="attention gqa causal", kind="attention", heads=32, kv_heads=8, tokens=32768, d=128, chunk=256, k=32,
             causal=True),
        # a short ragged prompt from tokens to attention output
        dict(name="prefill layer ragged", kind="prefill", heads=8, kv_heads=2, tokens=5003, d=64, chunk=48, k=12, m=6,
             r=6, causal=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng, most):
    kv = rng.choice([1, 2, 3, 4, 8, 8, 16, 32])
    group = rng.choice([1, 1, 2, 4])
    while kv * group > most:
        kv, group = max(1, kv // 2), max(1, group // 2)
    return kv * group, kv


def draw(rng):
    kind = rng.choice(["schedule"] * 6 + ["full"] * 2 + ["pool", "expand", "attention", "prefill"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if kind in ("schedule", "full"):
        heads, kv = _heads(rng, 32)
        n = _log(rng, 64, 2048)
        causal = rng.random() < 0.4
        nk = n if causal or rng.random() < 0.7 else _log(rng, 64, 2048)
        d = rng.choice([64, 128, 128, 32, 256] if dtype == "bf16" else [64, 128, 32])
        k = min(_log(rng, 8, 64), nk)
        budgets = rng.random() < 0.2
        if kind == "full":
            return dict(kind="full", heads=heads, kv_heads=kv, n=n, nk=nk, d=d, dtype=dtype, k=k, causal=causal,
                        budgets=budgets)
        m, r = rng.choice([k // 4, k // 2, k // 2, k]), rng.choice([k // 4, k // 2, k // 2])
        sinks, recent = rng.choice([(0, 0), (0, 0), (0, 0), (2, 2), (1, 4)])
        return _schedule("", heads, kv, n, nk, d, dtype, k, m, r, causal, round(10 ** rng.uniform(-2.3, -0.3), 4),
                         rng.randint(3, 8), rng.random() < 0.15, sinks, recent, rng.choice([0, 0, 0, 1]), budgets)
    heads, kv = _heads(rng, 32)
    if kind == "pool":
        d = rng.choice([32, 64, 128, 256])
        chunk = _log(rng, 16, 512)
        return dict(kind="pool", heads=heads, tokens=_log(rng, 512, 65536), d=d, chunk=chunk, dtype=dtype)
    chunk = _log(rng, 16, 256)
    k = _log(rng, 8, 48)
    causal = rng.random() < 0.7
    if kind == "expand":
        return dict(kind="expand", heads=heads, tokens=_log(rng, 1024, 32768), chunk=max(chunk, 32), k=k, causal=causal)
    tokens, d = _log(rng, 512, 16384), rng.choice([64, 128, 128])
    if kind == "attention":
        return dict(kind="attention", heads=heads, kv_heads=kv, tokens=tokens, d=d, chunk=chunk, k=k, causal=causal)
    # (the router takes up to 8192 chunks and k <= their number)
    k = min(k, -(-tokens // chunk))
    return dict(kind="prefill", heads=heads, kv_heads=kv, tokens=tokens, d=d, chunk=chunk, k=k, m=k // 2, r=k // 2,
                causal=causal)


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _layers(c, seed):
    """Chunk representations of every layer: clustered queries and keys that
    drift by an AR(1) step from layer to layer (the recipe of synth.py, drawn
    on the GPU)."""
    g = _gen(seed)
    heads, kv, n, nk, d = c["heads"], c["kv_heads"], c["n"], c["nk"], c["d"]
    rho, clusters = c.get("rho", 0.0), 64 if nk >= 512 else 16
    group = heads // kv
    randn = lambda *s: torch.randn(*s, generator=g, device=DEV)  # noqa: E731
    mu = randn(kv, clusters, d)
    zk = torch.randint(clusters, (kv, nk), generator=g, device=DEV)
    zq = torch.randint(clusters, (heads, n), generator=g, device=DEV)
    at = lambda mu, z: torch.gather(mu, 1, z[:, :, None].expand(-1, -1, d))  # noqa: E731
    K = (at(mu, zk) + 0.3 * randn(kv, nk, d)) / math.sqrt(d)
    Q = (at(mu.repeat_interleave(group, 0), zq) + 0.3 * randn(heads, n, d)) / math.sqrt(d)
    dup = src = None
    if c.get("near_ties"):
        order = torch.argsort(torch.rand(kv, nk, generator=g, device=DEV), dim=1)
        dup, src = order[:, :nk // 4], order[:, nk // 4:2 * (nk // 4)]
    out, keep = [], math.sqrt(1.0 - rho * rho)
    for layer in range(c.get("layers", 1)):
        if layer:
            Q = keep * Q + (rho / math.sqrt(d)) * randn(heads, n, d)
            K = keep * K + (rho / math.sqrt(d)) * randn(kv, nk, d)
        if dup is not None and dup.shape[1]:
            near = at(K, src) + 1e-3 * randn(kv, dup.shape[1], d)
            K = K.scatter(1, dup[:, :, None].expand(-1, -1, d), near)
        out.append((Q.to(_dtype(c["dtype"])).contiguous(), K.to(_dtype(c["dtype"])).contiguous()))
    return out


def _budgets(c, seed):
    """Per-row route widths: one of four buckets up to k per row."""
    if not c["budgets"]:
        return None
    widths = torch.tensor(sorted({max(1, c["k"] * q // 4) for q in (1, 2, 3, 4)}), dtype=torch.int32, device=DEV)
    return widths[torch.randint(len(widths), (c["heads"] * c["n"],), generator=_gen(seed + 7), device=DEV)].contiguous()


def _routes(c, seed):
    """Routes of a layer: every row takes its own chunk, the first chunk and
    other chunks at random, ids ascending, -1 padded."""
    nc, rows, k = -(-c["tokens"] // c["chunk"]), c["heads"] * -(-c["tokens"] // c["chunk"]), c["k"]
    g = _gen(seed + 3)
    s = torch.rand(rows, nc, generator=g, device=DEV)
    i = torch.arange(rows, device=DEV) % nc
    s[torch.arange(rows, device=DEV), i] = 2.0
    s[:, 0] = 3.0
    if c["causal"]:
        s.masked_fill_(torch.arange(nc, device=DEV)[None, :] > i[:, None], -1.0)
    take = min(k, nc)
    val, ids = torch.topk(s, take, dim=1)
    ids = torch.sort(torch.where(val >= 0, ids, nc), dim=1).values
    out = torch.full((rows, k), -1, dtype=torch.int32, device=DEV)
    out[:, :take] = torch.where(ids < nc, ids, -1).to(torch.int32)
    return out


def _tokens(c, heads, seed, dtype=torch.bfloat16):
    """Token vectors with a slowly changing mean (neighbouring tokens are
    alike, so that pooled chunks differ from one another)."""
    g = _gen(seed)
    n, d = c["tokens"], c["d"]
    coarse = torch.randn(heads, -(-n // 32), d, generator=g, device=DEV).repeat_interleave(32, 1)[:, :n]
    return (0.6 * coarse + 0.8 * torch.randn(heads, n, d, generator=g, device=DEV)).to(dtype).contiguous()


def _config(c, k_rows=None):
    return rr.Config(c["heads"], c["kv_heads"], c["n"], c["nk"], c["d"], c["k"], c.get("m", 0), c.get("r", 0),
                     c["dtype"], c["causal"], n_sink=c.get("sinks", 0), n_recent=c.get("recent", 0),
                     min_reuse=c.get("min_reuse", 0), k_rows=k_rows, seed=11)


def prepare(case, seed):
    c = case
    if c["kind"] == "schedule":
        cfg = _config(c, _budgets(c, seed))
        i32 = dict(dtype=torch.int32, device=DEV)
        return dict(
            kind="schedule", ledger=rr.Ledger(cfg), layers=_layers(c, seed),
            routes=[torch.empty(cfg.rows, cfg.k, **i32) for _ in range(c["layers"])],
            mask=[torch.empty(cfg.rows, dtype=torch.uint8, device=DEV) for _ in range(c["layers"] - 1)],
            pairs=[torch.empty(1, dtype=torch.int64, device=DEV) for _ in range(c["layers"])],
            rerouted=[torch.empty(1, **i32) for _ in range(c["layers"] - 1)])
    if c["kind"] == "full":
        cfg = _config(c, _budgets(c, seed))
        (Q, K), = _layers(c, seed)
        return dict(kind="full", cfg=cfg, Q=Q, K=K, routes=torch.empty(cfg.rows, cfg.k, dtype=torch.int32, device=DEV),
                    scores=torch.empty(cfg.rows, cfg.k, device=DEV),
                    pairs=torch.empty(1, dtype=torch.int64, device=DEV))
    if c["kind"] == "pool":
        X = _tokens(c, c["heads"], seed, _dtype(c["dtype"]))
        out = torch.empty(c["heads"], rr.n_chunks(c["tokens"], c["chunk"]), c["d"], dtype=X.dtype, device=DEV)
        return dict(kind="pool", X=X, chunk=c["chunk"], out=out)
    if c["kind"] == "expand":
        routes = _routes(c, seed)
        return dict(kind="expand", routes=routes, chunk=c["chunk"], tokens=c["tokens"],
                    out=torch.empty(routes.shape[0], c["k"] * c["chunk"], dtype=torch.int32, device=DEV))
    Q = _tokens(c, c["heads"], seed)
    K, V = _tokens(c, c["kv_heads"], seed + 1), _tokens(c, c["kv_heads"], seed + 2)
    s = dict(kind=c["kind"], Q=Q, K=K, V=V, chunk=c["chunk"], causal=c["causal"], out=torch.empty_like(Q))
    if c["kind"] == "attention":
        return dict(s, routes=_routes(c, seed))
    nc = rr.n_chunks(c["tokens"], c["chunk"])
    cfg = _config(dict(c, n=nc, nk=nc, dtype="bf16"))
    return dict(s, ledger=rr.Ledger(cfg), routes=torch.empty(cfg.rows, cfg.k, dtype=torch.int32, device=DEV))


def run(state):
    s = state
    if s["kind"] == "schedule":
        led = s["ledger"]
        for layer, (Q, K) in enumerate(s["layers"]):
            if layer == 0:
                led.anchor(0, Q, K, routes=s["routes"][0], pairs=s["pairs"][0])
            else:
                led.relay(layer, Q, K, routes=s["routes"][layer], mask=s["mask"][layer - 1], pairs=s["pairs"][layer],
                          n_rerouted=s["rerouted"][layer - 1])
        # (the counts are sums over the masks and ledgers returned: one row
        # whose boundary the last bit decides would change a whole output)
        return dict(routes=s["routes"], mask=s["mask"], ledger=led.export())
    if s["kind"] == "full":
        rr.full_route(s["cfg"], s["Q"], s["K"], s["routes"], scores=s["scores"], pairs=s["pairs"])
        return dict(routes=s["routes"], scores=s["scores"], pairs=s["pairs"])
    if s["kind"] == "pool":
        return rr.pool_chunks(s["X"], s["chunk"], out=s["out"])
    if s["kind"] == "expand":
        return rr.expand_tokens(s["routes"], s["chunk"], s["tokens"], out=s["out"])
    if s["kind"] == "attention":
        return rr.sparse_attention(s["Q"], s["K"], s["V"], s["routes"], s["chunk"], s["causal"], out=s["out"])
    Qc, Kc = rr.pool_chunks(s["Q"], s["chunk"]), rr.pool_chunks(s["K"], s["chunk"])
    s["ledger"].anchor(0, Qc, Kc, routes=s["routes"])
    O = rr.sparse_attention(s["Q"], s["K"], s["V"], s["routes"], s["chunk"], s["causal"], out=s["out"])
    return dict(Qc=Qc, Kc=Kc, routes=s["routes"], O=O)


# ---------------------------------------------------------- work, tolerance

def _pairs(c, n, nk):
    return c["heads"] * (n * (n + 1) // 2 if c["causal"] else n * nk)


def _route_bytes(c, n, nk):
    e = 2 if c.get("dtype", "bf16") == "bf16" else 4
    return (c["heads"] * n + c["kv_heads"] * nk) * c["d"] * e


def _attention_work(c):
    """Every token's routed keys (causal: half of the own chunk's); Q, K, V
    read once, O written once."""
    n, chunk, d = c["tokens"], c["chunk"], c["d"]
    nc = -(-n // chunk)
    keys = 0
    for i in range(nc):
        q = min(chunk, n - i * chunk)
        routed = min(c["k"], i + 1 if c["causal"] else nc)
        last = min(chunk, n - (nc - 1) * chunk)
        per = routed * chunk - (chunk // 2 if c["causal"] else 0) - (0 if c["causal"] else (chunk - last) * routed // nc)
        keys += q * max(per, 1)
    return dict(bytes=2 * d * n * 2 * (c["heads"] + c["kv_heads"]) + c["heads"] * nc * c["k"] * 4,
                flops=4 * d * keys * c["heads"])


def work(case):
    c = case
    if c["kind"] == "schedule":
        rows, c_led = c["heads"] * c["n"], c["k"] + c["m"] + c["r"] + c["sinks"] + c["recent"]
        pairs = _pairs(c, c["n"], c["nk"])
        # rows rerouted per relay layer: a fit of the measured shares over rho
        share = 1.0 - math.exp(-c["rho"] / 0.027)
        # per layer: inputs, the routes handed out, the mask; the ledger is
        # written and read once between layers
        per_layer = _route_bytes(c, c["n"], c["nk"]) + rows * (4 * c["k"] + 1) + 2 * rows * 4 * c_led
        return dict(bytes=c["layers"] * per_layer,
                    flops=2 * c["d"] * (pairs + (c["layers"] - 1) * (rows * min(c_led, c["nk"]) + share * pairs)))
    if c["kind"] == "full":
        return dict(bytes=_route_bytes(c, c["n"], c["nk"]) + 8 * c["heads"] * c["n"] * c["k"],
                    flops=2 * c["d"] * _pairs(c, c["n"], c["nk"]))
    if c["kind"] == "pool":
        e, nc = 2 if c["dtype"] == "bf16" else 4, -(-c["tokens"] // c["chunk"])
        return dict(bytes=c["heads"] * c["d"] * e * (c["tokens"] + nc), flops=c["heads"] * c["d"] * c["tokens"])
    if c["kind"] == "expand":
        rows = c["heads"] * -(-c["tokens"] // c["chunk"])
        return dict(bytes=4 * rows * c["k"] * (1 + c["chunk"]), flops=0)
    w = _attention_work(c)
    if c["kind"] == "attention":
        return w
    nc = -(-c["tokens"] // c["chunk"])
    pool = c["d"] * 2 * (c["heads"] + c["kv_heads"]) * (c["tokens"] + nc)
    return dict(bytes=w["bytes"] + pool + 4 * c["heads"] * nc * (c["k"] + c["m"] + c["r"]),
                flops=w["flops"] + 2 * c["d"] * _pairs(c, nc, nc))


def tolerance(case):
    # Measured as the difference of a pass from one on inputs whose features
    # (attention: route slots; pooling: tokens) are permuted, which is the same
    # result with its sums in another order, and stated about four times that:
    # route scores 1.5e-7 (largest 9e-7), ids 7e-6, pooled chunks 1.2e-7
    # (binary32; bf16: single roundings), attention 1.8e-3 (largest 0.02).
    # Routes are sets: where the order of a sum decides between two scores at a
    # row's boundary, the whole row's ids shift and its sentinels and the
    # layers after it follow, so a row or two in all may differ.
    c = case
    if c["kind"] == "expand":
        return "exact"
    if c["kind"] == "pool":
        return {"rel": 3e-5, "max": 8e-3} if c["dtype"] == "bf16" else {"rel": 5e-7, "max": 2e-6}
    if c["kind"] == "attention":
        return {"rel": 7e-3, "max": 0.08}
    if c["kind"] == "prefill":
        return {"rel": 7e-3, "max": 0.08, "differ": 3e-5 + 1.0 / (c["heads"] * -(-c["tokens"] // c["chunk"]))}
    rows = c["heads"] * c["n"]
    if c["kind"] == "full":
        return {"rel": 1e-5, "max": 1e-4, "differ": 3e-5 + 1.0 / rows}
    return {"rel": 0.0, "differ": min(0.01, 3e-5 + 2.0 / rows)}


# --------------------------------------------------------------------- exact

def _top(S, k, k_rows):
    """Rows' k best columns of S (higher first, equal: lower column), as ids
    ascending and their scores, -1 and -inf padded; -inf columns are invalid."""
    take = min(k, S.shape[1])
    val, ids = torch.sort(S, dim=1, descending=True, stable=True)
    val, ids = val[:, :take], ids[:, :take]
    keep = val > -math.inf
    if k_rows is not None:
        keep &= torch.arange(take, device=S.device)[None, :] < k_rows[:, None]
    big = S.shape[1]
    ids, order = torch.sort(torch.where(keep, ids, big), dim=1)
    val = torch.gather(val, 1, order)
    routes = torch.full((S.shape[0], k), -1, dtype=torch.int32, device=S.device)
    scores = torch.full((S.shape[0], k), -math.inf, dtype=torch.float64, device=S.device)
    routes[:, :take] = torch.where(ids < big, ids, -1).to(torch.int32)
    scores[:, :take] = torch.where(ids < big, val, -math.inf)
    return routes, scores


def _exact_routes(c, Q, K, k_rows=None):
    heads, n, nk = Q.shape[0], Q.shape[1], K.shape[1]
    group = heads // K.shape[0]
    routes, scores = [], []
    for h in range(heads):
        S = Q[h].double() @ K[h // group].double().t().contiguous()
        if c["causal"]:
            S.masked_fill_(torch.ones(n, nk, dtype=torch.bool, device=DEV).triu(1), -math.inf)
        r, s = _top(S, c["k"], None if k_rows is None else k_rows[h * n:(h + 1) * n])
        routes.append(r)
        scores.append(s)
    return torch.cat(routes), torch.cat(scores)


def _exact_pool(X, chunk):
    X = X.double()
    n = X.shape[1]
    whole = n // chunk
    parts = [X[:, :whole * chunk].reshape(X.shape[0], whole, chunk, X.shape[2]).mean(2)]
    if whole * chunk < n:
        parts.append(X[:, whole * chunk:].mean(1, keepdim=True))
    return torch.cat(parts, 1)


def _exact_attention(c, Q, K, V, routes):
    heads, n, d = Q.shape
    chunk, group = c["chunk"], heads // K.shape[0]
    nc = -(-n // chunk)
    K, V = K.double(), V.double()
    out = torch.zeros(heads, n, d, dtype=torch.float64, device=DEV)
    table = routes.cpu()
    inside = torch.arange(chunk, device=DEV)
    for h in range(heads):
        Kh, Vh = K[h // group], V[h // group]
        for i in range(nc):
            ids = table[h * nc + i]
            ids = ids[(ids >= 0) & (ids <= i)] if c["causal"] else ids[ids >= 0]
            if not len(ids):
                continue
            u = (ids.to(DEV)[:, None] * chunk + inside[None, :]).reshape(-1)
            u = u[u < n]
            t = torch.arange(i * chunk, min(n, (i + 1) * chunk), device=DEV)
            S = (Q[h, t].double() @ Kh[u].t().contiguous()) / math.sqrt(d)
            if c["causal"]:
                S.masked_fill_(u[None, :] > t[:, None], -math.inf)
            out[h, t] = torch.softmax(S, 1) @ Vh[u]
    return out


def exact(case, seed):
    c = case
    if c["kind"] == "schedule":
        # whole numbers only; after the anchor they follow from the ledger's
        # history, which has no value of its own in 64 bits
        Q, K = _layers(dict(c, layers=1), seed)[0]
        routes, _ = _exact_routes(c, Q, K, _budgets(c, seed))
        later = [None] * (c["layers"] - 1)
        return dict(routes=[routes] + later, mask=later, ledger=None)
    if c["kind"] == "full":
        (Q, K), = _layers(c, seed)
        routes, scores = _exact_routes(c, Q, K, _budgets(c, seed))
        return dict(routes=routes, scores=scores, pairs=torch.tensor([_pairs(c, c["n"], c["nk"])]))
    if c["kind"] == "pool":
        return _exact_pool(_tokens(c, c["heads"], seed, _dtype(c["dtype"])), c["chunk"])
    if c["kind"] == "expand":
        r = _routes(c, seed).long()
        u = r[:, :, None] * c["chunk"] + torch.arange(c["chunk"], device=DEV)
        return torch.where((r[:, :, None] >= 0) & (u < c["tokens"]), u, -1).reshape(r.shape[0], -1).to(torch.int32)
    Q = _tokens(c, c["heads"], seed)
    K, V = _tokens(c, c["kv_heads"], seed + 1), _tokens(c, c["kv_heads"], seed + 2)
    if c["kind"] == "attention":
        return _exact_attention(c, Q, K, V, _routes(c, seed))
    Qc, Kc = _exact_pool(Q, c["chunk"]), _exact_pool(K, c["chunk"])
    routes, _ = _exact_routes(c, Qc.to(torch.bfloat16), Kc.to(torch.bfloat16))
    return dict(Qc=Qc, Kc=Kc, routes=routes, O=_exact_attention(c, Q, K, V, routes))
