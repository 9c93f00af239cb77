"""Timed workloads over the range of uses of the search index.

Each case is one thing a program does with the library: it looks up queries in
an index it keeps, streams rows into one, puts a new database online, or runs
the exhaustive comparator.  Vectors are softmax features (softmax(z / T),
unit norm) as everywhere in this repository, with planted neighbours for some
queries; a "signed" index holds centred ones and a "clustered" one holds
groups of near duplicates.  Inputs are made on the device from the seed alone.
"""
import math

import torch

from paper_2311_02573_amd import gt

# kind       lookup    query() on a kept index
#            noalloc   query_noalloc(): the lookup in the library's fixed scratch
#            pipeline  three workspaces on three streams, one batch in each
#            exhaustive  the all-pairs comparator
#            stream    insert a group of rows, then query
#            build     build an index over the rows and answer the first batch
POOL_BYTES = {"f32": 4, "bf16": 2, "fp8": 1, "max_f32": 4, "max_bf16": 2}
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
STORE_BYTES = {"f32": 4, "f16": 2, "bf16": 2}
GROUP = 100        # rows of a streamed insert group
GROUPS = 64        # distinct groups a streaming program has at hand
WORKSPACES = 3     # batches in flight of a pipelined program
CLUSTERS, CLUSTER_ROWS = 8, 2000


def _case(kind, n, d, nq, pool="bf16", dtype="f32", rho=0.9, data="plain"):
    return {"kind": kind, "n": n, "d": d, "nq": nq, "pool": pool, "dtype": dtype, "rho": rho,
            "data": data}


def listed():
    named = {
        # one interactive lookup in a small collection: latency and launches only
        "one-small": _case("lookup", 16384, 128, 1),
        # one interactive lookup in the benchmark's database
        "one-1m": _case("lookup", 1 << 20, 1000, 1),
        # a handful of lookups on plain float32 pools, ragged in every size
        "ragged-f32": _case("lookup", 100003, 300, 65, pool="f32"),
        # a tight serving loop that must not allocate, float8 pools, ragged
        "noalloc-fp8": _case("noalloc", 300007, 777, 257, pool="fp8", dtype="f16", rho=0.8),
        # rows wider than the benchmark's, Our-Max pools
        "wide-max": _case("lookup", 1 << 17, 2048, 256, pool="max_bf16"),
        # the benchmark: batches of 1024 queries back to back on three workspaces
        "pipeline-1024": _case("pipeline", 1 << 20, 1000, 1024),
        # the benchmark's large batch on its smallest pools: the largest walk
        "batch-4096-fp8": _case("lookup", 1 << 20, 1000, 4096, pool="fp8"),
        # descriptors of any sign, the comparator's size
        "signed-1024": _case("lookup", 1 << 20, 512, 1024, pool="max_bf16", data="signed"),
        # near-duplicate clusters and per-query thresholds: long result lists
        "clustered": _case("lookup", 1 << 19, 256, 512, dtype="bf16", rho=0.0, data="clustered"),
        # the all-pairs comparator on the benchmark's database
        "exhaustive-1024": _case("exhaustive", 1 << 20, 1000, 1024),
        # the streaming setting: a query after every 100 inserted rows
        "stream-100": _case("stream", 1 << 20, 512, 16, dtype="f16"),
        # a new database with every sum format, and its first batch
        "build-200k": _case("build", 200000, 1000, 64),
    }
    return [dict(c, name=k) for k, c in named.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lookup"] * 6 + ["noalloc", "pipeline", "exhaustive", "stream", "build"])
    while True:
        n, d = _log_int(rng, 4096, 1 << 20), _log_int(rng, 100, 2048)
        nq = _log_int(rng, 1, 4096)
        if n * d > (1 << 20) * 1000 or n * nq / d > (1 << 20) * 4.096:
            continue
        if kind == "exhaustive" and n * nq * d > (1 << 30) * 1000:
            continue
        if kind == "pipeline" and nq > 1024:
            continue
        if kind == "stream" and (nq > 64 or n < 20000):
            continue
        if kind == "build" and (n * d > 200000 * 1000 or nq > 256):
            continue
        # the fixed scratch holds the query copies and a worst-case frontier
        # per query tile (64 queries, 32 for float32 pools)
        if kind == "noalloc" and nq * (12 * d + n) > (1 << 27):
            continue
        break
    data = "plain"
    pool = rng.choice(["bf16", "bf16", "fp8", "f32", "max_bf16"])
    if kind in ("lookup", "exhaustive"):
        data = rng.choice(["plain", "plain", "plain", "signed"])
        if kind == "lookup" and n >= 65536 and d <= 512 and nq >= 8 and rng.random() < 0.2:
            data = "clustered"
    if data == "signed":
        pool = "max_bf16"
    if kind in ("stream", "build"):
        pool = rng.choice(["bf16", "fp8"])
    rho = 0.0 if data == "clustered" else rng.choice([0.8, 0.9, 0.9, 0.95])
    return _case(kind, n, d, nq, pool=pool, dtype=rng.choice(["f32", "f32", "f16", "bf16"]),
                 rho=rho, data=data)


def _unit(z, temp, centred):
    x = torch.softmax(z / temp, dim=1)
    if centred:
        x -= 1.0 / x.shape[1]
    return x / x.norm(dim=1, keepdim=True)


def _inputs(case, seed):
    """(rows, queries, thresholds, streamed rows) of a case."""
    n, d = case["n"], case["d"]
    centred, clustered = case["data"] == "signed", case["data"] == "clustered"
    nq = case["nq"] * (WORKSPACES if case["kind"] == "pipeline" else 1)
    dev, store = torch.device("cuda"), DTYPES[case["dtype"]]
    g = torch.Generator(device=dev).manual_seed(seed)
    temp = 0.3 if clustered else 0.2 if d >= 512 else 0.25
    rows = torch.empty(n, d, dtype=store, device=dev)
    for a in range(0, n, 1 << 17):
        b = min(n, a + (1 << 17))
        rows[a:b] = _unit(torch.randn(b - a, d, device=dev, generator=g), temp, centred).to(store)
    qz = torch.randn(nq, d, device=dev, generator=g)
    rho = case["rho"]
    if clustered:
        centres = torch.randn(CLUSTERS, d, device=dev, generator=g)
        owner = torch.arange(CLUSTERS * CLUSTER_ROWS, device=dev) // CLUSTER_ROWS
        base, sigma, first = centres[owner], 0.02, max(1, nq // 10)
        pick = torch.randint(0, CLUSTERS, (first,), device=dev, generator=g)
        qz[:first] = centres[pick] + 0.02 * torch.randn(first, d, device=dev, generator=g)
        rho = (0.75 + 0.2 * torch.rand(nq, device=dev, generator=g, dtype=torch.float64)).cpu()
    else:
        # five planted neighbours a query on average; none in the streaming setting
        per = 0 if case["kind"] == "stream" else max(0, min(5, n // (2 * nq)))
        base, sigma = qz.repeat_interleave(per, dim=0), 0.05
    if base.shape[0]:
        at = torch.randperm(n, device=dev, generator=g)[: base.shape[0]]
        eps = sigma * torch.randn(base.shape, device=dev, generator=g)
        rows[at] = _unit(base + eps, temp, centred).to(store)
    extra = None
    if case["kind"] == "stream":
        extra = _unit(torch.randn(GROUP * GROUPS, d, device=dev, generator=g), temp, False).to(store)
    return rows, _unit(qz, temp, centred), rho, extra


def _matches(case):
    """About how many rows match one query of a case's data."""
    clustered = 0.1 * CLUSTER_ROWS if case["data"] == "clustered" else 0
    return min(case["n"], 5 + clustered + 0.25 * case["n"] / case["d"])


def _table_rows(case):
    """Room for one batch's results."""
    return 1024 + int(4 * case["nq"] * _matches(case))


def _pools(case):
    if case["data"] == "signed":
        return ("signed", "max_bf16")
    if case["kind"] == "build":
        return ("f32", "bf16", "fp8")
    return ("f32", case["pool"])


def prepare(case, seed):
    rows, q, rho, extra = _inputs(case, seed)
    rho = rho if isinstance(rho, float) else rho.numpy()
    s = {"case": case, "q": q, "rho": rho}
    kind, room = case["kind"], _table_rows(case)
    s["tables"] = [(torch.zeros(room, dtype=torch.int64, device="cuda"),
                    torch.zeros(room, dtype=torch.float32, device="cuda"))
                   for _ in range(WORKSPACES if kind == "pipeline" else 1)]
    if kind == "build":
        s["rows"] = rows
        return s
    if kind == "stream":
        s["rows"], s["extra"], s["next"] = rows, extra, 0
        s["capacity"] = 1 << (case["n"] + (1 << 18)).bit_length()
        s["index"] = gt.GTIndex(rows, capacity=s["capacity"], pools=_pools(case))
        return s
    s["index"] = gt.GTIndex(rows, pools=_pools(case))
    if kind == "pipeline":
        s["batches"] = list(q.split(case["nq"]))
        s["workspaces"] = [gt.Workspace(s["index"], case["nq"]) for _ in range(WORKSPACES)]
    return s


def _out(s, r, k=0):
    """The results in the program's own table k (ids and cosines end to end,
    by query; what lies past the last result is not the call's)."""
    ids, sims = s["tables"][k]
    t = min(r.total, ids.shape[0])
    ids[:t].copy_(r.ids[:t])
    sims[:t].copy_(r.sims[:t])
    return {"offsets": r.offsets, "ids": ids, "sims": sims}


def run(s):
    case = s["case"]
    kind, pool = case["kind"], case["pool"]
    if kind == "lookup":
        return _out(s, s["index"].query(s["q"], s["rho"], pool=pool))
    if kind == "noalloc":
        return _out(s, s["index"].query_noalloc(s["q"], s["rho"], pool=pool))
    if kind == "exhaustive":
        return _out(s, s["index"].exhaustive(s["q"], s["rho"]))
    if kind == "pipeline":
        for ws, q in zip(s["workspaces"], s["batches"]):
            ws.submit(q, s["rho"], pool=pool)
        return [_out(s, ws.finish(), k) for k, ws in enumerate(s["workspaces"])]
    if kind == "stream":
        if s["index"].n + GROUP > s["capacity"]:  # full: start over from the first rows
            s["index"].close()
            s["index"] = gt.GTIndex(s["rows"], capacity=s["capacity"], pools=_pools(case))
        k = s["next"]
        s["next"] = (k + 1) % GROUPS
        first = s["index"].insert(s["extra"][k * GROUP : (k + 1) * GROUP])
        return {"first": first, **_out(s, s["index"].query(s["q"], s["rho"], pool=pool))}
    index = gt.GTIndex(s["rows"], pools=_pools(case))
    out = _out(s, index.query(s["q"], s["rho"], pool=pool))
    index.close()
    return out


def work(case):
    """What a pass cannot do without.  A search has to look at every part of
    the tree once (here: the pools of 16 rows, in the walked format) and test
    every match exactly on its float32 row; about 0.25 n / d of the rows match
    a query of this data, beside its planted neighbours."""
    n, d = case["n"], case["d"]
    nq = case["nq"] * (WORKSPACES if case["kind"] == "pipeline" else 1)
    matches = nq * _matches(case)
    io = nq * (4 * d + 8) + 12 * matches
    if case["kind"] == "exhaustive":
        return {"bytes": 4 * n * d + io, "flops": 2 * n * d * nq}
    width = 2 * d if case["data"] == "signed" else d
    search = n / 16 * width * POOL_BYTES[case["pool"]] + 4 * d * min(n, matches) + io
    flops = 2 * nq * width * n / 16 + 2 * d * matches
    store = STORE_BYTES[case["dtype"]]
    if case["kind"] == "stream":
        # the inserted rows in and out, and their paths' pools rewritten
        path = 4 + POOL_BYTES[case["pool"]]
        search += GROUP * d * (store + 4) + 2 * GROUP * d * path
    if case["kind"] == "build":
        # rows in, leaves and the pools of every format out
        search += n * d * (store + 4 + 4 + 2 + 1)
        flops += n * d
    return {"bytes": search, "flops": flops}


def _exact_lookup(rows, q, rho, room):
    """Range search by float64 products: offsets, ids and cosines."""
    nq = q.shape[0]
    q64 = q.double()
    q64 = q64 / q64.norm(dim=1, keepdim=True)
    lim = torch.as_tensor(rho, dtype=torch.float64, device=q.device).expand(nq)
    found = []
    for a in range(0, rows.shape[0], 1 << 16):
        f64 = rows[a : a + (1 << 16)].double()
        cos = q64 @ (f64 / f64.norm(dim=1, keepdim=True)).t()
        hit = (cos >= lim[:, None]).nonzero()
        found.append((hit[:, 0], hit[:, 1] + a, cos[hit[:, 0], hit[:, 1]]))
    owner, ids, sims = (torch.cat(x) for x in zip(*found))
    order = torch.argsort(owner, stable=True)
    counts = torch.bincount(owner, minlength=nq)
    offsets = torch.zeros(nq + 1, dtype=torch.int64, device=q.device)
    offsets[1:] = counts.cumsum(0)
    table = (torch.zeros(room, dtype=torch.int64, device=q.device),
             torch.zeros(room, dtype=torch.float64, device=q.device))
    t = min(room, ids.shape[0])
    table[0][:t], table[1][:t] = ids[order][:t], sims[order][:t]
    return {"offsets": offsets, "ids": table[0], "sims": table[1]}


def exact(case, seed):
    rows, q, rho, extra = _inputs(case, seed)
    room = _table_rows(case)
    if case["kind"] == "pipeline":
        return [_exact_lookup(rows, b, rho, room) for b in q.split(case["nq"])]
    if case["kind"] == "stream":
        rows = torch.cat([rows, extra[:GROUP]])
        return {"first": case["n"], **_exact_lookup(rows, q, rho, room)}
    return _exact_lookup(rows, q, rho, room)
