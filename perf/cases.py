"""Workloads of the dynamic Leiden library that its speed is judged by.

Each case is one call sequence of a user's program through the public Python
interface (``paper_2405_11658_amd.leiden``): streamed batch updates of a
resident graph, clustering of a graph just loaded, a fleet of small graphs,
several graphs updated at once, and the single steps that can be called by
themselves (aggregation, modularity, marking).

Graphs.  The R-MAT graphs are the ones of ``inputs.rmat_device`` (edge factor
16, as the repository's benchmark).  The asynchronous sweeps of the default
mode may end in different partitions from run to run on a graph without clear
communities, so the cases in that mode use weighted similarity graphs: planted
communities of heavy-tailed degrees (vertex ids permuted) with edges of weight
1 inside and weak edges anywhere.  Their partition is unambiguous, however the
sweep's timing falls.  Labels follow the timing all the same, so a community
is named by its smallest member, as a program does that follows communities
from one update to the next.
"""
from __future__ import annotations

import math

import torch

from paper_2405_11658_amd import inputs as gen
from paper_2405_11658_amd import leiden as L

DEV = "cuda"
EDGE_FACTOR = 16


# ---- cases -------------------------------------------------------------------
def listed():
    return [
        # the smallest streamed update: 4096 vertices (the planted graphs of the
        # tests have this size), about a hundred changed edges
        {"name": "update_df_4k", "kind": "update", "n": 4096, "mode": "df", "frac": 1e-3},
        # an ordinary graph under a stream of DF batches of 1e-4 |E|, the
        # benchmark's batch size
        {"name": "update_df_500k", "kind": "update", "n": 524288, "mode": "df", "frac": 1e-4},
        # Delta-screening, which marks whole communities; vertex count a prime
        {"name": "update_ds_1m", "kind": "update", "n": 1000003, "mode": "ds", "frac": 1e-4},
        # the largest: 8.4M vertices, about 220M directed entries
        {"name": "update_df_8m", "kind": "update", "n": 8388608, "mode": "df", "frac": 1e-4},
        # several mid-sized resident graphs updated by one call
        {"name": "many_nd_16", "kind": "many", "graphs": 16, "nmin": 2000, "nmax": 60000, "mode": "nd", "frac": 1e-3},
        # a graph loaded and clustered from scratch
        {"name": "static_1m", "kind": "static", "n": 1048576, "sync": False},
        # the same in the reproducible mode, on an R-MAT graph (heavy hubs, no
        # clear communities), vertex count odd
        {"name": "static_sync_rmat17", "kind": "static", "n": 100003, "sync": True},
        # a handful of small graphs, and the 512 of 1e3 .. 3e4 vertices of the
        # repository's many-graph experiment
        {"name": "fleet_24", "kind": "fleet", "graphs": 24, "nmin": 500, "nmax": 4000, "mode": "df", "frac": 3e-3},
        {"name": "fleet_512", "kind": "fleet", "graphs": 512, "nmin": 1000, "nmax": 30000, "mode": "df", "frac": 3e-3},
        # single steps: super-vertex graph of a weighted R-MAT graph, modularity
        # of a membership, marking of a batch (which stages the graph update)
        {"name": "aggregate_rmat21", "kind": "aggregate", "n": 2097152},
        {"name": "modularity_rmat22", "kind": "modularity", "n": 4194304},
        {"name": "mark_df_rmat20", "kind": "mark", "n": 1048573, "mode": "df", "frac": 1e-3},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _logf(rng, lo, hi):
    return float("%.3g" % math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["update", "update", "update", "many", "static", "fleet", "aggregate", "modularity", "mark"])
    mode = rng.choice(["df", "df", "nd", "ds"])
    if kind == "update":
        return {"kind": kind, "n": _log(rng, 2000, 6000000), "mode": mode, "frac": _logf(rng, 1e-5, 3e-3)}
    if kind == "many":
        return {"kind": kind, "graphs": rng.randint(3, 24), "nmin": 2000, "nmax": _log(rng, 4000, 60000), "mode": mode,
                "frac": _logf(rng, 1e-4, 3e-3)}
    if kind == "static":
        sync = rng.random() < 0.3
        return {"kind": kind, "n": _log(rng, 2000, 100000 if sync else 2000000), "sync": sync}
    if kind == "fleet":
        return {"kind": kind, "graphs": _log(rng, 8, 512), "nmin": 500, "nmax": _log(rng, 1000, 30000),
                "mode": rng.choice(["df", "nd", "ds", "static"]), "frac": _logf(rng, 1e-3, 1e-2)}
    if kind == "aggregate":
        return {"kind": kind, "n": _log(rng, 2000, 2097152)}
    if kind == "modularity":
        return {"kind": kind, "n": _log(rng, 2000, 4194304)}
    return {"kind": kind, "n": _log(rng, 2000, 1500000), "mode": mode, "frac": _logf(rng, 1e-5, 1e-2)}


# ---- inputs ------------------------------------------------------------------
PICKS = 9        # uniform neighbours drawn per vertex inside its community
HEAVY = 6.0      # heavy-tailed edge ends per vertex inside communities
CROSS = 3.0      # heavy-tailed edge ends per vertex anywhere in its graph
WEAK = 2.0 ** -10  # weight of an edge between communities (similarity graphs)


def _communities(n):
    """Communities of a similarity graph: few enough that their weights stay far
    above modularity's resolution limit."""
    return max(8, int(math.sqrt(n) / 4))


def _planted(g, sizes):
    """Edges (u, v) of vertices lying in communities of the given consecutive
    sizes, PICKS uniform and HEAVY / 2 heavy-tailed ones per vertex inside
    them, the community of each vertex, and the function that draws heavy-tailed
    vertices."""
    n, k = int(sizes.sum()), sizes.numel()
    f64 = torch.float64
    start = torch.cumsum(sizes, 0) - sizes
    com = torch.repeat_interleave(torch.arange(k, device=DEV), sizes)
    r = torch.rand(n, generator=g, device=DEV, dtype=f64)
    # whole numbers: their sums do not depend on the order they are taken in
    theta = (1024 * torch.clamp((1 - r) ** (-1 / 1.5), max=max(2.0, n / k / 8))).long()
    cum = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    cum[1:] = torch.cumsum(theta, 0)

    def heavy(lo, hi):  # a vertex of the id range [lo, hi), by weight
        x = cum[lo] + (torch.rand(lo.numel(), generator=g, device=DEV, dtype=f64) * (cum[hi] - cum[lo])).long()
        return torch.minimum(torch.clamp(torch.searchsorted(cum, x, right=True) - 1, min=0), hi - 1)

    u0 = torch.arange(n, device=DEV).repeat_interleave(PICKS)
    c0 = com[u0]
    v0 = start[c0] + (torch.rand(u0.numel(), generator=g, device=DEV, dtype=f64) * sizes[c0]).long()
    u1 = heavy(*_range(int(n * HEAVY / 2), n))
    v1 = heavy(start[com[u1]], (start + sizes)[com[u1]])
    return torch.cat([u0, u1]), torch.cat([v0, v1]), com, heavy


def _range(m, n):
    z = torch.zeros(m, dtype=torch.int64, device=DEV)
    return z, z + n


def _keys(n, u, v):
    keep = u != v
    u, v = u[keep], v[keep]
    return torch.unique(torch.cat([u * n + v, v * n + u]))


def _csr(n, key):
    off = torch.searchsorted(key, torch.arange(n + 1, device=DEV) * n)
    idx = (key % n).to(torch.int32)
    return off, idx, torch.ones(idx.numel(), dtype=torch.float32, device=DEV)


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _similarity(n, seed):
    """One planted graph: (off, idx, w) and the community of each vertex."""
    g = _generator(seed)
    k = _communities(n)
    sizes = torch.full((k,), n // k, device=DEV)
    sizes[: n % k] += 1
    u, v, com, heavy = _planted(g, sizes)
    a, b = heavy(*_range(int(n * CROSS / 2), n)), heavy(*_range(int(n * CROSS / 2), n))
    perm = torch.randperm(n, generator=g, device=DEV)
    label = torch.empty(n, dtype=torch.int32, device=DEV)
    label[perm] = com.to(torch.int32)
    key = _keys(n, perm[torch.cat([u, a])], perm[torch.cat([v, b])])
    off, idx, _ = _csr(n, key)
    return (off, idx, _weight(label, key // n, idx)), label


def _weight(label, u, v):
    return torch.where(label[u.long()] == label[v.long()], 1.0, WEAK).to(torch.float32)


def _batch(n, off, idx, label, frac, seed):
    """A batch of frac |E| random updates (four in five of them insertions) of
    a planted graph, and the batch that takes it back."""
    du, dv, iu, iv, _ = gen.batch_stream_device(n, off, idx, gen.batch_count(idx.numel(), frac), 1, seed=seed + 1)[0]
    there, new = _weight(label, du, dv), _weight(label, iu, iv)
    return (du, dv, iu, iv, new), (iu, iv, du, dv, there)


def _rmat(n, seed):
    return gen.rmat_device(max(1, math.ceil(math.log2(n))), EDGE_FACTOR, seed=seed, n=n)[1:]


def _sizes(case):
    """Vertex counts of a case of several graphs, spread over the logarithm."""
    lo, hi, k = math.log(case["nmin"]), math.log(case["nmax"]), case["graphs"]
    return [int(round(math.exp(lo + (hi - lo) * ((37 * j + 11) % k + 0.5) / k))) for j in range(k)]


def _undo(b):  # of a batch of unit weights
    return b[2], b[3], b[0], b[1], torch.ones(b[0].numel(), dtype=torch.float32, device=DEV)


def _fleet(case, seed):
    """The graphs of a fleet (communities of about 64 vertices, one edge in
    five between them) and a batch for each, drawn together: the graphs are
    the diagonal blocks of one big one."""
    g = _generator(seed)
    ns = _sizes(case)
    sizes, owner = [], []
    for j, n in enumerate(ns):
        k = max(1, n // 64)
        sizes += [n // k + (1 if q < n % k else 0) for q in range(k)]
        owner += [j] * k
    sizes, owner = torch.tensor(sizes, device=DEV), torch.tensor(owner, device=DEV)
    n = int(sizes.sum())
    u, v, com, heavy = _planted(g, sizes)
    graph = owner[com]
    a = heavy(*_range(int(n * CROSS), n))
    ends = torch.cumsum(torch.tensor(ns, device=DEV), 0)
    b = heavy((ends - torch.tensor(ns, device=DEV))[graph[a]], ends[graph[a]])
    u, v = torch.cat([u, a]), torch.cat([v, b])
    count = torch.tensor(ns, device=DEV)
    base = torch.cumsum(count, 0) - count
    # vertex ids permuted inside each graph
    perm = torch.empty(n, dtype=torch.int64, device=DEV)
    perm[torch.argsort(graph + torch.rand(n, generator=g, device=DEV, dtype=torch.float64))] = torch.arange(n, device=DEV)
    key = _keys(n, perm[u], perm[v])
    off, idx, w = _csr(n, key)
    idx = (idx - base[graph[key // n]].to(torch.int32)).contiguous()
    ends = torch.cat([base, count.sum().reshape(1)])
    cuts, rows = off[ends].tolist(), ends.tolist()
    graphs = [(off[rows[j]: rows[j + 1] + 1] - cuts[j], idx[cuts[j]: cuts[j + 1]], w[cuts[j]: cuts[j + 1]])
              for j in range(len(ns))]
    if case["mode"] == "static":
        return graphs, None
    # batches: frac of each graph's entries, four in five of them insertions
    m = int(key.numel() * case["frac"] * 2)
    a = torch.randint(0, n, (m,), generator=g, device=DEV)
    ga = graph[a]
    b = base[ga] + (torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * count[ga]).long()
    ins = torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))
    at = torch.clamp(torch.searchsorted(key, ins), max=key.numel() - 1)
    ins = ins[(key[at] != ins) & (ins // n != ins % n)]
    ins = ins[torch.rand(ins.numel(), generator=g, device=DEV) < 0.4]
    one_way = key[key // n < key % n]
    old = one_way[torch.rand(one_way.numel(), generator=g, device=DEV) < 0.4 * case["frac"]]
    batches = []
    ci = torch.searchsorted(ins // n, ends).tolist()
    co = torch.searchsorted(old // n, ends).tolist()
    iu, iv = (ins // n), (ins % n)
    du, dv = (old // n), (old % n)
    for j in range(len(ns)):
        i, o, z = slice(ci[j], ci[j + 1]), slice(co[j], co[j + 1]), rows[j]
        t = [(x - z).to(torch.int32) for x in (du[o], dv[o], iu[i], iv[i])]
        batches.append((*t, torch.ones(ci[j + 1] - ci[j], dtype=torch.float32, device=DEV)))
    return graphs, batches


def _membership(n, off, idx, seed):
    """Dense labels of clusters grown along edges, as a first level's are:
    every vertex points to one of its neighbours, chains followed to depth 4."""
    g = _generator(seed)
    deg = off[1:] - off[:-1]
    pick = off[:-1] + (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * deg).long()
    own = torch.arange(n, device=DEV)
    to = torch.where(deg > 0, idx[torch.clamp(pick, max=idx.numel() - 1)].long(), own)
    to = torch.minimum(to, own)
    to = to[to]
    to = to[to]
    label, inverse = torch.unique(to, return_inverse=True)
    return inverse.to(torch.int32), label.numel()


def _weighted(n, seed):
    """A weighted R-MAT graph and a membership.  One graph for each size, its
    vertices, labels and weights shuffled by the seed, so that its super-vertex
    graph has the same number of entries for every seed."""
    off, idx, _ = _rmat(n, 1)
    label, count = _membership(n, off, idx, 2)
    g = _generator(seed)
    to = torch.randperm(n, generator=g, device=DEV)
    name = torch.randperm(count, generator=g, device=DEV)
    off, idx, _ = _csr(n, torch.sort(to[_rows(n, off)] * n + to[idx.long()])[0])
    moved = torch.empty_like(label)
    moved[to] = name[label.long()].to(torch.int32)
    return (off, idx, 0.25 + torch.rand(idx.numel(), generator=g, device=DEV)), moved, count


def prepare(case, seed):
    kind = case["kind"]
    if kind == "update":
        n = case["n"]
        (off, idx, w), label = _similarity(n, seed)
        h = L.leiden_create(off, idx, w)
        L.leiden_set_state(h, label)  # the membership that the stream so far has left
        b, undo = _batch(n, off, idx, label, case["frac"], seed)
        return {"kind": kind, "h": h, "mode": case["mode"], "batches": (b, undo)}
    if kind == "many":
        hs, bs, us = [], [], []
        for j, n in enumerate(_sizes(case)):
            (off, idx, w), label = _similarity(n, seed * 1000 + j)
            h = L.leiden_create(off, idx, w)
            L.leiden_set_state(h, label)
            b, undo = _batch(n, off, idx, label, case["frac"], seed * 1000 + j)
            hs.append(h)
            bs.append(b)
            us.append(undo)
        return {"kind": kind, "hs": hs, "modes": [case["mode"]] * len(hs), "batches": (bs, us)}
    if kind == "static":
        graph = _rmat(case["n"], seed) if case["sync"] else _similarity(case["n"], seed)[0]
        return {"kind": kind, "graph": graph, "params": L.leiden_default_params(sync_mode=int(case["sync"])),
                "sync": case["sync"]}
    if kind == "fleet":
        graphs, batches = _fleet(case, seed)
        fleet = L.Fleet(graphs)
        k = len(graphs)
        static = [(j, "static", None) for j in range(k)]
        if batches is None:
            return {"kind": kind, "fleet": fleet, "runs": (static,)}
        fleet.run(static, want_membership=False)
        return {"kind": kind, "fleet": fleet,
                "runs": ([(j, case["mode"], batches[j]) for j in range(k)],
                         [(j, case["mode"], _undo(batches[j])) for j in range(k)])}
    n = case["n"]
    if kind == "mark":
        off, idx, w = _rmat(n, seed)
        h = L.leiden_create(off, idx, w)
        L.leiden_set_state(h, _membership(n, off, idx, seed)[0])
        b = gen.batch_stream_device(n, off, idx, gen.batch_count(idx.numel(), case["frac"]), 1, seed=seed)[0]
        return {"kind": kind, "h": h, "mode": case["mode"], "batch": b}
    graph, label, count = _weighted(n, seed)
    return {"kind": kind, "graph": graph, "label": label, "count": count}


# ---- one pass ------------------------------------------------------------------
def _named(C):
    """Communities named by their smallest member."""
    n = C.numel()
    own = torch.arange(n, device=C.device)
    label, order = torch.sort(C, stable=True)
    head = torch.ones(n, dtype=torch.bool, device=C.device)
    head[1:] = label[1:] != label[:-1]
    low = torch.empty(2 * n, dtype=torch.int64, device=C.device)
    low.scatter_(0, torch.where(head, label.long(), own + n), order)
    return low[C.long()]


def run(state):
    kind = state["kind"]
    if kind == "update":
        # a batch arrives, and later its changes are taken back
        h, out = state["h"], []
        for b in state["batches"]:
            C, q, _, _ = L.leiden_update(h, b, state["mode"])
            out += [_named(C), q]
        C, K, S, m2 = L.leiden_get_state(h)
        return {"update": out, "K": K, "community_weight": S[C.long()], "m2": m2}
    if kind == "many":
        out = []
        for bs in state["batches"]:
            done = L.leiden_update_many(state["hs"], bs, state["modes"])
            out += [torch.cat([_named(C) for C, _, _, _ in done]), [q for _, q, _, _ in done],
                    max(status for _, _, _, status in done)]
        return out
    if kind == "static":
        h = L.leiden_create(*state["graph"], state["params"])
        C, q, _ = L.leiden_static(h)
        L.leiden_destroy(h)
        return C if state["sync"] else _named(C), q
    if kind == "fleet":
        out = []
        for jobs in state["runs"]:
            done, _ = state["fleet"].run(jobs)
            out += [torch.cat([C for C, _, _, _ in done]), torch.tensor([q for _, q, _, _ in done], dtype=torch.float64),
                    max(status for _, _, status, _ in done)]
        return out
    if kind == "aggregate":
        return L.leiden_aggregate(*state["graph"], state["label"], state["count"])
    if kind == "modularity":
        return L.leiden_modularity(*state["graph"], state["label"])
    return L.leiden_mark_affected(state["h"], state["batch"], state["mode"])


# ---- what a pass cannot do without ---------------------------------------------
def _entries(n):
    return int(n * (2 * PICKS + HEAVY + CROSS) * 0.98)


def work(case):
    kind = case["kind"]
    graph = lambda n, nnz: 8 * (n + 1) + 8 * nnz  # noqa: E731
    if kind in ("update", "many", "fleet"):
        # per update: the old graph read, the new one written, the batch, the
        # state read and written and the membership
        total = flops = 0
        passes = 1 if case["mode"] == "static" else 2
        for n in [case["n"]] if kind == "update" else _sizes(case):
            nnz = _entries(n) if kind != "fleet" else int(n * (2 * PICKS + HEAVY + 2 * CROSS) * 0.8)
            total += passes * (passes * graph(n, nnz) + 24 * gen.batch_count(nnz, case["frac"]) + 44 * n)
            flops += passes * 4 * nnz
        return {"bytes": total, "flops": flops}
    n = case["n"]
    if kind == "static":
        nnz = 30 * n if case["sync"] else _entries(n)
        return {"bytes": 2 * graph(n, nnz) + 24 * n, "flops": 4 * nnz}
    nnz = int(29.5 * n)
    if kind == "aggregate":  # about three in four entries stay distinct pairs
        return {"bytes": graph(n, nnz) + 4 * n + int(0.75 * graph(n, nnz)), "flops": nnz}
    if kind == "modularity":
        return {"bytes": graph(n, nnz) + 4 * n, "flops": 2 * nnz}
    return {"bytes": 2 * graph(n, nnz) + 24 * gen.batch_count(nnz, case["frac"]) + 23 * n, "flops": nnz}


# ---- reference values in 64 bits -------------------------------------------------
def _q(n, src, dst, w, C):
    """(Eq. 1, K, Sigma of every vertex's community, 2m) in float64."""
    w = w.double()
    K = torch.zeros(n, dtype=torch.float64, device=DEV).scatter_add_(0, src, w)
    S = torch.zeros(n, dtype=torch.float64, device=DEV).scatter_add_(0, C, K)
    m2 = float(w.sum())
    inside = float(w[C[src] == C[dst]].sum())
    return inside / m2 - float(((S / m2) ** 2).sum()), K, S[C], m2


def _rows(n, off):
    return torch.repeat_interleave(torch.arange(n, device=DEV), off[1:] - off[:-1])


def exact(case, seed):
    kind = case["kind"]
    n = case.get("n")
    if kind == "update":
        (off, idx, w), label = _similarity(n, seed)
        b = _batch(n, off, idx, label, case["frac"], seed)[0]
        C = label.long()
        key = _rows(n, off) * n + idx.long()
        du, dv, iu, iv = (x.long() for x in b[:4])
        gone = torch.searchsorted(key, torch.cat([du * n + dv, dv * n + du]))
        w1 = w.clone()
        w1[gone] = 0.0
        src, dst = torch.cat([key // n, iu, iv]), torch.cat([idx.long(), iv, iu])
        q1 = _q(n, src, dst, torch.cat([w1, b[4], b[4]]), C)[0]
        q0, K, S, m2 = _q(n, key // n, idx.long(), w, C)
        return {"update": [None, q1, None, q0], "K": K, "community_weight": S, "m2": m2}
    if kind == "static" and not case["sync"]:
        (off, idx, w), label = _similarity(n, seed)
        return None, _q(n, _rows(n, off), idx.long(), w, label.long())[0]
    if kind == "modularity":
        (off, idx, w), label, _ = _weighted(n, seed)
        return _q(n, _rows(n, off), idx.long(), w, label.long())[0]
    if kind == "aggregate":
        (off, idx, w), label, count = _weighted(n, seed)
        C = label.long()
        pair, inverse = torch.unique(C[_rows(n, off)] * count + C[idx.long()], return_inverse=True)
        total = torch.zeros(pair.numel(), dtype=torch.float64, device=DEV).scatter_add_(0, inverse, w.double())
        return (torch.searchsorted(pair, torch.arange(count + 1, device=DEV) * count), (pair % count).to(torch.int32),
                total)
    return None
