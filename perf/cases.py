"""Performance cases of the library: what a program that uses it has it do,
through its public entry points, over the range of sizes and options that the
tests and the benchmark of this repository use.

Kinds of case:

  sssp     one single-source query.  api "plain": sssp() with its defaults
           (parDijkstra, one extraction per round).  api "learned": sssp_ex()
           with the trained extraction threshold and the settings that the
           autotuner picks on such graphs (bulk size d, team, k_max, k_every,
           deep-level workers).  api "noalloc": sssp_noalloc(), the entry of
           callers that must not allocate.  api "nearfar": the Delta-stepping
           baseline.
  batch    many queries in one launch: sssp_batch(), plain or learned.
  heap     a priority queue in steady state on either engine: rounds of
           bulk_update (decrease-keys and insertions, some ids twice), delete
           and extract_min, the times moving forward with the extracted keys
           as in an event simulation or a best-first search.
  train    Adam steps on the threshold model: mlp_train().

Graphs are the repository's families (4- and 8-neighbour grids, ring
lattices, random geometric graphs, the paper's high-diameter DAG), built on
the GPU from the seed.
"""
import math

import torch

import paper_1908_09378_amd as pkg
from paper_1908_09378_amd import learn

DEV = "cuda:0"
FAR = 1 << 62


def listed():
    return [
        # The repository's small configuration: one query on a 64 x 64 street
        # grid, default options.  4,096 dependent rounds with d = 4.
        {"name": "plain_grid4_64", "kind": "sssp", "api": "plain", "graph": "grid4", "rows": 64, "cols": 64},
        # A long, narrow network (the ring lattice of the benchmark, shorter):
        # default options, d = 32, a frontier of a few hundred vertices.
        {"name": "plain_ring_12k", "kind": "sssp", "api": "plain", "graph": "ring", "n": 12289, "k": 16},
        # The paper's own workload, a dense high-diameter DAG, at a fifth of
        # its vertices and half of its mean degree: d in the thousands, the
        # top bucket in HBM, rows of a thousand edges.
        {"name": "plain_dag_6k", "kind": "sssp", "api": "plain", "graph": "dag", "n": 6000, "deg": 1000},
        # The comparison family on a terrain grid: Near-Far (Delta-stepping),
        # default delta, some hundred phases over the whole device.
        {"name": "nearfar_grid8_401", "kind": "sssp", "api": "nearfar", "graph": "grid8", "rows": 401, "cols": 397},
        # The headline: the learned threshold on a ring lattice, tuned settings.
        {"name": "learned_ring_100k", "kind": "sssp", "api": "learned", "graph": "ring", "n": 100003, "k": 16,
         "d": 128, "team": 256, "k_max": 256, "k_every": 16, "deep": 0},
        # The large-heap form: an 8-neighbour terrain grid with log-uniform
        # weights, deep-level workers.
        {"name": "learned_grid8_361", "kind": "sssp", "api": "learned", "graph": "grid8", "rows": 361, "cols": 359,
         "d": 256, "team": 256, "k_max": 256, "k_every": 4, "deep": 2},
        # Many queries at once over graphs of uneven size (random geometric,
        # mean degree 24, four sources each), learned threshold, tuned.
        {"name": "batch_rgg_learned", "kind": "batch", "rule": "learned", "graph": "rgg", "graphs": 24, "sources": 4,
         "lo": 4096, "hi": 65536, "d_scale": 32, "team": 256, "k_max": 256},
        # Many small plain queries at once over ring lattices and grids: what
        # the training pipeline runs to collect its traces.
        {"name": "batch_mixed_plain", "kind": "batch", "rule": "plain", "graph": "mixed", "graphs": 64, "sources": 2,
         "lo": 300, "hi": 4096, "d_scale": 0, "team": 0, "k_max": 0},
        # The standalone heap at the benchmark's size: 2^24 ids, bulk updates
        # of 2^20, extracts of 2^16, device-wide engine.
        {"name": "heap_wide_16m", "kind": "heap", "ids": 1 << 24, "d": 1 << 20, "batch": 1 << 20, "take": 1 << 16,
         "drop": 0, "rounds": 4},
        # A mid-size heap on the device-wide engine, deletes among the
        # operations, odd sizes.
        {"name": "heap_wide_1m", "kind": "heap", "ids": 1000003, "d": 50021, "batch": 40009, "take": 5003,
         "drop": 1201, "rounds": 4},
        # A small heap on the one-workgroup engine: each call is a few short
        # kernels and the host's calls around them.
        {"name": "heap_team_10k", "kind": "heap", "ids": 10007, "d": 256, "batch": 256, "take": 60, "drop": 9,
         "rounds": 4},
        # Training of the threshold model: Adam steps on batches of 1,024.
        {"name": "train_1024", "kind": "train", "samples": 16384, "batch": 1024, "steps": 16},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "learned", "learned", "nearfar", "noalloc", "batch", "batch", "heap", "heap",
                       "train"])
    if kind in ("plain", "nearfar"):
        graph = rng.choice(["grid4", "grid8", "ring", "dag"] if kind == "plain" else ["grid4", "grid8", "ring"])
        c = {"kind": "sssp", "api": kind, "graph": graph}
        top = 9000 if kind == "plain" else 200000
        if graph == "dag":
            n = _log(rng, 600, 6000)
            c.update(n=n, deg=rng.randint(8, min(1000, n // 5)))
        elif graph == "ring":
            c.update(n=_log(rng, 80, top), k=rng.choice([3, 8, 16]))
        else:
            n = _log(rng, 64, min(top, 5000) if kind == "plain" else top)
            rows = max(2, int(math.sqrt(n) * rng.uniform(0.5, 1.0)))
            c.update(rows=rows, cols=max(2, n // rows))
        return c
    if kind in ("learned", "noalloc"):
        graph = rng.choice(["grid4", "grid8", "ring"])
        c = {"kind": "sssp", "api": kind, "graph": graph}
        n = _log(rng, 400, 60000 if kind == "learned" else 4000)
        if graph == "ring":
            c.update(n=n, k=16)
        else:
            rows = max(2, int(math.sqrt(n) * rng.uniform(0.5, 1.0)))
            c.update(rows=rows, cols=max(2, n // rows))
        d = rng.choice([64, 128, 256])
        deep = rng.choice([0, 0, 2]) if kind == "learned" else 0
        c.update(d=d, team=rng.choice([64, 256]) if kind == "learned" else 64, k_max=rng.choice([64, 256]),
                 k_every=rng.choice([1, 4, 16]), deep=deep)
        return c
    if kind == "batch":
        if rng.random() < 0.5:
            lo = _log(rng, 500, 8000)
            return {"kind": "batch", "rule": "learned", "graph": "rgg", "graphs": rng.randint(3, 20),
                    "sources": rng.randint(1, 4), "lo": lo, "hi": min(50000, lo * rng.randint(2, 10)),
                    "d_scale": rng.choice([8, 16, 32]), "team": 256, "k_max": 256}
        lo = _log(rng, 100, 600)
        return {"kind": "batch", "rule": "plain", "graph": "mixed", "graphs": rng.randint(3, 100),
                "sources": rng.randint(1, 3), "lo": lo, "hi": min(3500, lo * rng.randint(2, 8)), "d_scale": 0,
                "team": 0, "k_max": 0}
    if kind == "heap":
        wide = rng.random() < 0.6
        d = _log(rng, 16384, 600000) if wide else _log(rng, 32, 3000)
        ids = int(d * rng.uniform(3, 14 if wide else 40)) | 1
        batch = max(8, int(d * rng.uniform(0.3, 1.0)))
        take = max(2, int(batch * rng.uniform(0.02, 0.25)))
        return {"kind": "heap", "ids": ids, "d": d, "batch": batch, "take": take,
                "drop": rng.choice([0, max(1, batch // 40)]), "rounds": 4}
    batch = _log(rng, 100, 2048)
    return {"kind": "train", "samples": batch * rng.randint(2, 12) + rng.randint(0, batch - 1), "batch": batch,
            "steps": rng.randint(4, 16)}


# ------------------------------------------------------------------- graphs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _loguniform(g, count):
    u = torch.rand(count, generator=g, device=DEV, dtype=torch.float64)
    return torch.exp(u * math.log(10001.0)).floor().clamp(1, 10000).to(torch.int64)


def _csr(n, src, dst, w):
    """Rows sorted by target."""
    order = torch.argsort(src * n + dst, stable=True)
    counts = torch.bincount(src, minlength=n)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(counts, 0, out=off[1:])
    return off, dst[order].to(torch.int32), w[order].to(torch.int32), n


def _undirected(n, a, b, w):
    return _csr(n, torch.cat([a, b]), torch.cat([b, a]), torch.cat([w, w]))


def _grid(g, rows, cols, eight):
    ids = torch.arange(rows * cols, device=DEV).view(rows, cols)
    pairs = [(ids[:, :-1], ids[:, 1:]), (ids[:-1], ids[1:])]
    if eight:
        pairs += [(ids[:-1, :-1], ids[1:, 1:]), (ids[:-1, 1:], ids[1:, :-1])]
    a = torch.cat([p[0].reshape(-1) for p in pairs])
    b = torch.cat([p[1].reshape(-1) for p in pairs])
    w = _loguniform(g, a.numel()) if eight else torch.randint(1, 101, (a.numel(),), generator=g, device=DEV)
    return _undirected(rows * cols, a, b, w)


def _ring(g, n, k):
    i = torch.arange(n, device=DEV).view(n, 1)
    j = torch.arange(1, k + 1, device=DEV).view(1, k)
    a = i.expand(n, k).reshape(-1)
    b = ((i + j) % n).reshape(-1)
    return _undirected(n, a, b, torch.randint(1, 1001, (n * k,), generator=g, device=DEV))


def _dag(g, n, deg):
    """Chain edges of weight 1 and random forward edges of weight 2 (v - u),
    so that dist(i) = i - s from vertex s; about n * deg edges."""
    tails = torch.arange(n, device=DEV).view(n, 1)
    heads = torch.arange(n, device=DEV).view(1, n)
    room = (n - 2 - tails).clamp(min=1)
    p = (deg * 1.0 / room).clamp(max=1.0)
    pick = (torch.rand(n, n, generator=g, device=DEV) < p) & (heads > tails + 1)
    pick |= heads == tails + 1
    e = pick.nonzero()
    src, dst = e[:, 0], e[:, 1]
    gap = dst - src
    w = torch.where(gap == 1, gap, 2 * gap)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(pick.sum(1), 0, out=off[1:])
    return off, dst.to(torch.int32), w.to(torch.int32), n


def _rgg(g, n):
    """n points in the unit square, edges below the radius of mean degree 24,
    weight round(1000 length) + 1; points binned in cells of that radius."""
    r = math.sqrt(24.0 / (math.pi * n))
    side = max(1, int(1.0 / r))
    xy = torch.rand(n, 2, generator=g, device=DEV, dtype=torch.float64)
    cell = (xy * side).long().clamp(max=side - 1)
    cid = cell[:, 0] * side + cell[:, 1]
    order = torch.argsort(cid, stable=True)
    starts = torch.searchsorted(cid[order], torch.arange(side * side + 1, device=DEV))
    cs = cell[order]
    srcs, dsts, ws = [], [], []
    for dx in (-1, 0, 1):
        for dy in (-1, 0, 1):
            nx, ny = cs[:, 0] + dx, cs[:, 1] + dy
            at = ((nx >= 0) & (nx < side) & (ny >= 0) & (ny < side)).nonzero().view(-1)
            nc = nx[at] * side + ny[at]
            lo = starts[nc]
            cnt = starts[nc + 1] - lo
            rep = torch.repeat_interleave(at, cnt)
            first = torch.repeat_interleave(lo - (torch.cumsum(cnt, 0) - cnt), cnt)
            cand = first + torch.arange(rep.numel(), device=DEV)
            a, b = order[rep], order[cand]
            dd = (xy[a] - xy[b]).square().sum(1)
            keep = (dd < r * r) & (a != b)
            srcs.append(a[keep])
            dsts.append(b[keep])
            ws.append((1000.0 * dd[keep].sqrt()).round().long() + 1)
    return _csr(n, torch.cat(srcs), torch.cat(dsts), torch.cat(ws))


def _graph(case, g):
    if case["graph"] == "ring":
        return _ring(g, case["n"], case["k"])
    if case["graph"] == "dag":
        return _dag(g, case["n"], case["deg"])
    return _grid(g, case["rows"], case["cols"], case["graph"] == "grid8")


def _sizes(case):
    """The vertex counts of a batch's graphs, spread evenly over the
    logarithm of the case's range."""
    n = case["graphs"]
    step = math.log(case["hi"] / case["lo"]) / max(1, n - 1)
    return [int(case["lo"] * math.exp(step * i)) for i in range(n)]


def _batch_graphs(case, g):
    out = []
    for i, n in enumerate(_sizes(case)):
        if case["graph"] == "rgg":
            out.append(_rgg(g, n))
        elif i % 3 == 0:
            out.append(_ring(g, max(n, 40), 16))
        else:
            side = max(3, int(math.sqrt(n)))
            out.append(_grid(g, side, side, i % 3 == 2))
    return out


def _source(case, seed):
    # a DAG is entered near its head; the vertices before the source stay
    # unreached
    return int(seed) % (1 + case["n"] // 50) if case["graph"] == "dag" else 0


def _batch_sources(case, seed, graphs):
    host = torch.Generator().manual_seed(int(seed) + 1)
    return [[int(x) for x in torch.randint(0, gr[3], (case["sources"],), generator=host)] for gr in graphs]


def _model():
    return torch.from_numpy(learn.load_model()).to(DEV)


# --------------------------------------------------------------------- heap
def _heap_inputs(case, seed):
    g = _gen(seed)
    n = case["ids"]
    keys = torch.randint(0, 1 << 40, (n,), generator=g, device=DEV)
    # ids of the updates: every id in random order, one in 16 replaced by a
    # random one, so that some ids come twice and some batches hold duplicates
    pool = torch.randperm(n, generator=g, device=DEV).to(torch.int32)
    pool[::16] = torch.randint(0, n, (pool[::16].numel(),), generator=g, device=DEV).to(torch.int32)
    later = torch.randint(1, 1 << 40, (n,), generator=g, device=DEV)
    gone = torch.randint(0, n, (max(1, 16 * case["drop"]),), generator=g, device=DEV).to(torch.int32)
    return keys, pool, later, gone


class _HeapState:
    def __init__(self, case, seed):
        self.case = case
        keys, self.pool, self.later, self.gone = _heap_inputs(case, seed)
        n, d, k = case["ids"], case["d"], case["take"]
        self.heap = pkg.Heap(n, d)
        ids = torch.arange(n, device=DEV, dtype=torch.int32)
        for at in range(0, n, d):
            self.heap.bulk_update(keys[at:at + d].contiguous(), ids[at:at + d].contiguous())
        self.keys = torch.empty(case["batch"], dtype=torch.int64, device=DEV)
        self.ko = [torch.empty(k, dtype=torch.int64, device=DEV) for _ in range(case["rounds"])]
        self.io = [torch.empty(k, dtype=torch.int32, device=DEV) for _ in range(case["rounds"])]
        self.heap.extract_min(k, self.ko[-1], self.io[-1])
        self.at = self.cut = 0


def _next(at, count, total):
    """Where the next `count` of a pool of `total` entries start."""
    return at if at + count <= total else 0


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    if case["kind"] == "heap":
        return _HeapState(case, seed)
    g = _gen(seed)
    if case["kind"] == "train":
        n = case["samples"]
        X = torch.randn(n, 8, generator=g, device=DEV) * 3.0 + 5.0
        X[:, 5] *= 0.125
        # labels as the traces give them: log2 of a pull size that grows with
        # the heap and shrinks with the key spread, between 0 and 5
        Y = (0.8 * X[:, 1] - 0.4 * X[:, 2] + 1.5 + torch.randn(n, generator=g, device=DEV)).clamp(0, 5)
        start = torch.from_numpy(learn.init_blob(int(seed) & 0xFFFF)).to(DEV)
        pkg.mlp_feature_stats(X, start)
        return {"case": case, "X": X, "Y": Y, "start": start}
    if case["kind"] == "batch":
        graphs = _batch_graphs(case, g)
        queries = []
        for (off, tg, wt, n), srcs in zip(graphs, _batch_sources(case, seed, graphs)):
            for s in srcs:
                queries.append((off, tg, wt, n, tg.numel(), s, torch.empty(n, dtype=torch.int64, device=DEV)))
        opts = {}
        if case["rule"] == "learned":
            opts = dict(k_rule=pkg.K_LEARNED, k_model=_model(), d_scale=case["d_scale"], team=case["team"],
                        k_max=case["k_max"])
        return {"case": case, "queries": queries, "opts": opts}
    off, tg, wt, n = _graph(case, g)
    args = (off, tg, wt, n, tg.numel(), _source(case, seed), torch.empty(n, dtype=torch.int64, device=DEV))
    opts = {}
    if case["api"] in ("learned", "noalloc"):
        opts = dict(k_rule=pkg.K_LEARNED, k_model=_model(), d=case["d"], team=case["team"], k_max=case["k_max"],
                    k_every=case["k_every"], deep_level=case["deep"])
    return {"case": case, "args": args, "opts": opts}


# ---------------------------------------------------------------------- run
def run(state):
    if isinstance(state, _HeapState):
        return _run_heap(state)
    case = state["case"]
    if case["kind"] == "train":
        blob = state["start"].clone()
        losses = pkg.mlp_train(state["X"], state["Y"], blob, case["batch"], case["steps"], 1e-3)
        return blob, losses
    if case["kind"] == "batch":
        pkg.sssp_batch(state["queries"], **state["opts"])
        # one tensor: the queries' distances one after another
        return torch.cat([q[6] for q in state["queries"]])
    a = state["args"]
    if case["api"] == "plain":
        pkg.sssp(*a)
    elif case["api"] == "nearfar":
        pkg.sssp_nearfar(*a)
    elif case["api"] == "noalloc":
        pkg.sssp_noalloc(*a, **state["opts"])
    else:
        pkg.sssp_ex(*a, **state["opts"])
    return a[6]


def _run_heap(s):
    c = s.case
    n, b, k, drop = c["ids"], c["batch"], c["take"], c["drop"]
    now = s.ko[-1][k - 1:]
    got = []
    for r in range(c["rounds"]):
        s.at = _next(s.at, b, n)
        # updates lie ahead of the last extracted key
        torch.add(s.later[s.at:s.at + b], now, out=s.keys)
        s.heap.bulk_update(s.keys, s.pool[s.at:s.at + b])
        s.at += b
        if drop:
            s.cut = _next(s.cut, drop, s.gone.numel())
            s.heap.delete(s.gone[s.cut:s.cut + drop])
            s.cut += drop
        got.append(s.heap.extract_min(k, s.ko[r], s.io[r]))
        now = s.ko[r][k - 1:]
    return got, s.ko, s.io, s.heap.size()


# --------------------------------------------------------------------- work
def _edges(case):
    if case["graph"] == "ring":
        return case["n"], 2 * case["k"] * case["n"]
    if case["graph"] == "dag":
        return case["n"], case["n"] * case["deg"]
    r, c = case["rows"], case["cols"]
    m = 2 * (r * (c - 1) + (r - 1) * c)
    if case["graph"] == "grid8":
        m += 4 * (r - 1) * (c - 1)
    return r * c, m


def work(case):
    """Every input read once, every output written once: a query's offsets,
    targets, weights and distances, a heap call's pairs and ids, the training
    samples and the model."""
    if case["kind"] == "sssp":
        n, m = _edges(case)
        return {"bytes": 8 * (n + 1) + 8 * m + 8 * n, "flops": 0}
    if case["kind"] == "batch":
        total = 0
        for i, n in enumerate(_sizes(case)):
            deg = 24 if case["graph"] == "rgg" else (32, 4, 8)[i % 3]
            total += 8 * n + 8 * deg * n + 8 * n * case["sources"]
        return {"bytes": total, "flops": 0}
    if case["kind"] == "heap":
        return {"bytes": case["rounds"] * (12 * case["batch"] + 12 * case["take"] + 4 * case["drop"]), "flops": 0}
    seen = case["steps"] * min(case["batch"], case["samples"])
    params = 8 * 64 + 64 * 64 + 64
    return {"bytes": min(seen, case["samples"]) * 36 + 8 * pkg.MLP_BLOB, "flops": 6 * params * seen}


def tolerance(case):
    if case["kind"] != "train":
        return "exact"
    return {"rel": 2e-4}


# -------------------------------------------------------------------- exact
def _bellman_ford(off, tg, wt, n, source):
    """Distances by relaxing every edge until nothing changes (int64)."""
    src = torch.repeat_interleave(torch.arange(n, device=DEV), off[1:] - off[:-1])
    dst, w = tg.long(), wt.long()
    dist = torch.full((n,), FAR, dtype=torch.int64, device=DEV)
    dist[source] = 0
    while True:
        before = dist.clone()
        for _ in range(32):
            dist.scatter_reduce_(0, dst, dist[src] + w, "amin")
        if torch.equal(before, dist):
            break
    return torch.where(dist >= FAR, torch.full_like(dist, -1), dist)


def _exact_heap(case, seed):
    keys, pool, later, gone = _heap_inputs(case, seed)
    n, b, k, drop = case["ids"], case["batch"], case["take"], case["drop"]
    cur = keys.clone()

    def take():
        order = torch.sort(cur, stable=True)  # equal keys stay in id order
        ids = order.indices[:k]
        cur[ids] = FAR
        return order.values[:k].clone(), ids.to(torch.int32)

    now = take()[0][-1]
    at = cut = 0
    got, ko, io = [], [], []
    for _ in range(case["rounds"]):
        at = _next(at, b, n)
        cur.scatter_reduce_(0, pool[at:at + b].long(), later[at:at + b] + now, "amin")
        at += b
        if drop:
            cut = _next(cut, drop, gone.numel())
            cur[gone[cut:cut + drop].long()] = FAR
            cut += drop
        a, i = take()
        got.append(k)
        ko.append(a)
        io.append(i)
        now = a[-1]
    return got, ko, io, int((cur < FAR).sum())


def _exact_train(case, seed):
    s = prepare(case, seed)
    X, Y, blob = s["X"].double(), s["Y"].double(), s["start"].double()
    batch = min(case["batch"], case["samples"])
    mu, sd = blob[pkg.MLP_PARAMS:pkg.MLP_PARAMS + 8], blob[pkg.MLP_PARAMS + 8:pkg.MLP_PARAMS + 16]
    w = blob[:pkg.MLP_PARAMS].clone()
    m, v = torch.zeros_like(w), torch.zeros_like(w)
    losses = []
    for t in range(case["steps"]):
        at = (t % (case["samples"] // batch)) * batch
        x, y = (X[at:at + batch] - mu) / sd, Y[at:at + batch]
        # the forward pass uses the weights rounded to bfloat16; the rounding
        # is taken as identity in the backward pass
        p = w.to(torch.bfloat16).double().requires_grad_(True)
        w1, b1, w2, b2, w3, b3 = torch.split(p, [512, 64, 4096, 64, 64, 1])
        h = torch.nn.functional.gelu(x @ w1.view(8, 64) + b1)
        h = torch.nn.functional.gelu(h @ w2.view(64, 64) + b2)
        loss = ((h @ w3 + b3 - y) ** 2).mean()
        (grad,) = torch.autograd.grad(loss, p)
        losses.append(float(loss))
        m = 0.9 * m + 0.1 * grad
        v = 0.999 * v + 0.001 * grad * grad
        w = w - 1e-3 * (m / (1 - 0.9 ** (t + 1))) / ((v / (1 - 0.999 ** (t + 1))).sqrt() + 1e-8)
    blob[:pkg.MLP_PARAMS] = w.to(torch.bfloat16).double()
    return blob, torch.tensor(losses, dtype=torch.float64).numpy()


def exact(case, seed):
    if case["kind"] == "heap":
        return _exact_heap(case, seed)
    if case["kind"] == "train":
        return _exact_train(case, seed)
    g = _gen(seed)
    if case["kind"] == "batch":
        graphs = _batch_graphs(case, g)
        out = []
        for (off, tg, wt, n), srcs in zip(graphs, _batch_sources(case, seed, graphs)):
            out += [_bellman_ford(off, tg, wt, n, s) for s in srcs]
        return torch.cat(out)
    off, tg, wt, n = _graph(case, g)
    if case["graph"] == "dag":
        return (torch.arange(n, device=DEV) - _source(case, seed)).clamp(min=-1)
    return _bellman_ford(off, tg, wt, n, 0)
