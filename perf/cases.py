"""Measured cases: hypergraphs kept on the GPU and updated in batches.

A case names its path (`kind`) and its sizes; `prepare` makes the hypergraph and
the update batches from a seed and builds the resident graph(s), `run` is one
step of a program that keeps triad counts up to date: it applies one batch
through a public entry point and reads the counts.

Steps can be repeated on one state.  A vertical batch deletes the hyperedges
that the step before inserted (the first one: uniformly chosen ones) and inserts
as many; two insert sets take turns, so the graph keeps its size.  A temporal
batch replaces the oldest arrivals, with timestamps that move on.  Horizontal
operations are undone by the next step.

Every output is a whole number (assigned IDs, exact 64-bit counts).
"""
import itertools
import math

import numpy as np
import torch

from paper_2512_21009_amd import hgt

HE_IV = "hyperedge+incident_vertex"
ALL = "hyperedge+incident_vertex+temporal"


# --------------------------------------------------------------------------- #
# the cases
# --------------------------------------------------------------------------- #
def _medium(scale):
    """The benchmark's Medium shape at a scale: cardinality power law 2.5 on [2, 64],
    vertex popularity (rank + 10^4 scale)^-1.1, two hyperedges per vertex."""
    return dict(nv=max(64, round(1_000_000 * scale)), ne=max(16, round(2_000_000 * scale)), alpha=2.5, lo=2, hi=64,
                s=1.1, q=1.0e4 * scale)


def _arrivals(scale):
    """The benchmark's Temporal shape at a scale: uniform popularity, power law 2.2
    on [2, 128], arrivals over one hour of expiry, window 600 s."""
    return dict(nv=max(256, round(500_000 * scale)), alpha=2.2, lo=2, hi=128, s=0.0, q=0.0,
                gap_us=1000.0 / scale, window_us=600_000_000)


def listed():
    return [
        # one changed hyperedge in a small resident graph, scratch never allocated:
        # an online service that applies every event as it comes (pure latency)
        dict(name="single_update", kind="batch", changes=1, track=HE_IV, noalloc=True, **_medium(0.01)),
        # the repository's Tiny workload: hub-heavy small hypergraph, 100 + 100 changes
        dict(name="tiny_batch", kind="batch", changes=100, track=HE_IV, noalloc=False,
             nv=2000, ne=1000, alpha=0.0, lo=2, hi=8, s=1.2, q=0.0),
        # an ordinary update of an ordinary graph: 2,500 + 2,500 changes on 500k hyperedges
        dict(name="ordinary_batch", kind="batch", changes=2_500, track=HE_IV, noalloc=False, **_medium(0.25)),
        # the headline workload at full size: 50k + 50k changes on 2M hyperedges
        dict(name="medium_batch", kind="batch", changes=50_000, track=HE_IV, noalloc=False, **_medium(1.0)),
        # a small event stream that keeps all three families at once
        dict(name="stream_all", kind="stream", ne=36_000, batch=2_000, track=ALL, **_arrivals(0.01)),
        # the temporal stream at a quarter of its full size: 50k arrivals replace the oldest 50k
        dict(name="stream_temporal", kind="stream", ne=900_000, batch=50_000, track="temporal", **_arrivals(0.25)),
        # a plain graph (every hyperedge an edge): triangle counting under 100k edge changes
        dict(name="dyadic_batch", kind="dyadic", nv=1_000_000, ne=8_000_000, s=0.8, q=1.0e3, changes=50_000),
        # the paper's scaling sweep (|V| = |E| / 3, uniform, heavy tail of cardinalities)
        dict(name="large_random", kind="batch", changes=25_000, track="hyperedge", noalloc=False,
             nv=6_666_666, ne=20_000_000, alpha=3.0, lo=2, hi=1024, s=0.0, q=0.0),
        # many independent hypergraphs updated by one call, sizes and batches log-uniform
        dict(name="batched_graphs", kind="batched", graphs=48, e_lo=1_000, e_hi=100_000, b_lo=10, b_hi=20_000, hi=256,
             graph=False),
        # many small hypergraphs whose round is launched as one HIP graph
        dict(name="batched_small", kind="batched", graphs=64, e_lo=500, e_hi=4_000, b_lo=10, b_hi=100, hi=32, graph=True),
        # the request server: every tenant sends one request from host memory, all families kept
        dict(name="served_round", kind="served", tenants=16, total=60_000, b_lo=2, b_hi=400, hi=64, q=150.0),
        # horizontal operations: vertices enter and leave live hyperedges
        dict(name="vertex_ops", kind="vertex_ops", ops=25_000, track=HE_IV, **_medium(0.25)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a path by its weight in use, its sizes log-uniform over the listed range."""
    kind = rng.choice(["batch", "batch", "batch", "stream", "stream", "dyadic", "batched", "served", "vertex_ops"])
    if kind == "batch":
        c = _medium(_log_int(rng, 1_000, 500_000) / 1e6)
        c["hi"] = rng.choice([8, 32, 64, 100])
        c["s"] = rng.choice([0.0, 0.8, 1.1])
        return dict(kind=kind, changes=_log_int(rng, 1, max(2, c["ne"] // 40)), noalloc=False,
                    track=rng.choice([HE_IV, HE_IV, "hyperedge", "incident_vertex"]), **c)
    if kind == "stream":
        scale = _log_int(rng, 5_000, 150_000) / 1e6
        ne = round(3_600_000 * scale)
        return dict(kind=kind, ne=ne, batch=_log_int(rng, max(2, ne // 200), ne // 18),
                    track=rng.choice(["temporal", "hyperedge+temporal", ALL]), **_arrivals(scale))
    if kind == "dyadic":
        ne = _log_int(rng, 10_000, 3_000_000)
        return dict(kind=kind, nv=max(2000, ne // rng.randint(4, 12)), ne=ne, s=rng.choice([0.0, 0.5, 0.8]), q=1.0e3,
                    changes=_log_int(rng, 1, ne // 100))
    if kind == "batched":
        b_hi = _log_int(rng, 50, 5_000)
        return dict(kind=kind, graphs=rng.randint(2, 60), e_lo=500, e_hi=_log_int(rng, 2_000, 50_000), b_lo=2, b_hi=b_hi,
                    hi=rng.choice([16, 64, 256]), graph=rng.random() < 0.5)
    if kind == "served":
        tenants = rng.randint(2, 24)
        return dict(kind=kind, tenants=tenants, total=tenants * _log_int(rng, 1_000, 4_000), b_lo=2,
                    b_hi=_log_int(rng, 20, 400), hi=64, q=150.0)
    c = _medium(_log_int(rng, 1_000, 250_000) / 1e6)
    return dict(kind=kind, ops=_log_int(rng, 2, max(4, c["ne"] // 20)), track=rng.choice([HE_IV, "hyperedge"]), **c)


# --------------------------------------------------------------------------- #
# inputs (made on the GPU from the seed alone)
# --------------------------------------------------------------------------- #
DEV = "cuda"


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


class _Vertices:
    """Popularity (rank + q)^-s over nv vertices; ranks map to ids by a permutation."""

    def __init__(self, g, nv, s, q):
        self.g, self.nv = g, nv
        self.perm = torch.randperm(nv, generator=g, device=DEV)
        self.cdf = None
        if s:
            w = (torch.arange(1, nv + 1, dtype=torch.float64, device=DEV) + q) ** -s
            self.cdf = torch.cumsum(w, 0)
            self.cdf = self.cdf / self.cdf[-1].clone()

    def draw(self, n):
        if self.cdf is None:
            r = torch.randint(self.nv, (n,), generator=self.g, device=DEV)
        else:
            r = torch.searchsorted(self.cdf, torch.rand(n, generator=self.g, device=DEV, dtype=torch.float64), right=True)
            r = r.clamp_(max=self.nv - 1)
        return self.perm[r]


def _cards(g, n, alpha, lo, hi):
    """Cardinalities from P(k) ~ k^-alpha on [lo, hi] (alpha 0: uniform)."""
    w = torch.arange(lo, hi + 1, dtype=torch.float64, device=DEV) ** -alpha
    cdf = torch.cumsum(w, 0)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * cdf[-1]
    return (lo + torch.searchsorted(cdf, u, right=True)).clamp_(max=hi)


def _rows(g, cards, vert):
    """(offsets int64, members int32) of rows of distinct vertices in random order."""
    n, nv = len(cards), vert.nv
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(cards, 0, out=off[1:])
    row = torch.repeat_interleave(torch.arange(n, device=DEV), cards)
    key = row * nv + vert.draw(len(row))
    while True:  # draw repeated vertices of a row again
        key = key.sort().values
        dup = torch.zeros(len(key), dtype=torch.bool, device=DEV)
        dup[1:] = key[1:] == key[:-1]
        at = dup.nonzero().flatten()
        if not len(at):
            break
        key[at] = row[at] * nv + vert.draw(len(at))
    order = (row << 31 | torch.randint(1 << 31, (len(row),), generator=g, device=DEV)).argsort()
    return off, (key[order] % nv).to(torch.int32)


def _split(off, mem, a, b):
    """Rows [a, b) of a CSR as a CSR of their own."""
    lo, hi = off[[a, b]].tolist()
    return off[a:b + 1] - lo, mem[lo:hi].clone()


def _make_rows(c, seed, n):
    g = _gen(seed)
    vert = _Vertices(g, c["nv"], c["s"], c["q"])
    return g, vert, _rows(g, _cards(g, n, c["alpha"], c["lo"], min(c["hi"], c["nv"] // 4)), vert)


def _batch_inputs(c, seed):
    """(initial CSR, deleted IDs, two insert CSRs) of a vertical case."""
    ne, n = c["ne"], c["changes"]
    if c["kind"] == "dyadic":
        g = _gen(seed)
        vert = _Vertices(g, c["nv"], c["s"], c["q"])
        want, key = ne + 2 * n, torch.zeros(0, dtype=torch.int64, device=DEV)
        while len(key) < want:  # distinct edges
            ends = vert.draw(2 * (want + want // 8 + 16)).view(-1, 2)
            lo, hi = ends.min(1).values, ends.max(1).values
            key = torch.unique(torch.cat([key, (lo * c["nv"] + hi)[lo != hi]]))
        key = key[torch.randperm(len(key), generator=g, device=DEV)[:want]]
        mem = torch.stack([key // c["nv"], key % c["nv"]], 1)
        flip = torch.rand(want, generator=g, device=DEV) < 0.5
        mem = torch.where(flip[:, None], mem.flip(1), mem).flatten().to(torch.int32)
        off = 2 * torch.arange(want + 1, device=DEV)
    else:
        g, _, (off, mem) = _make_rows(c, seed, ne + 2 * n)
    dels = torch.randperm(ne, generator=g, device=DEV)[:n].to(torch.int32)
    return _split(off, mem, 0, ne), dels, [_split(off, mem, ne + k * n, ne + (k + 1) * n) for k in range(2)]


def _track(c):
    return tuple(c["track"].split("+"))


def _prepare_batch(c, seed):
    c = dict(c, track=c.get("track", "incident_vertex"))
    (off, mem), dels, sets = _batch_inputs(c, seed)
    graph = hgt.Graph.build(c["nv"], off, mem, track=_track(c))
    return dict(kind="batch", graph=graph, track=_track(c), noalloc=c.get("noalloc", False), ids=dels,
                turn=itertools.cycle(sets))


def _arrival_times(g, n, gap_us):
    gaps = torch.empty(n, dtype=torch.float64, device=DEV).exponential_(1.0 / gap_us, generator=g)
    return torch.cumsum(gaps.floor().to(torch.int64), 0)


def _prepare_stream(c, seed):
    ne, n = c["ne"], c["batch"]
    g, _, (off, mem) = _make_rows(c, seed, ne)
    ts = _arrival_times(g, ne, c["gap_us"])
    graph = hgt.Graph.build(c["nv"], off, mem, ts, track=_track(c), window=c["window_us"])
    slots = []  # consecutive runs of n arrivals: the oldest run leaves, its successor of the same content arrives
    for a in range(0, ne - n + 1, n):
        o, m = _split(off, mem, a, a + n)
        slots.append(dict(ids=torch.arange(a, a + n, dtype=torch.int32, device=DEV), off=o, mem=m, ts=ts[a:a + n].clone()))
    return dict(kind="stream", graph=graph, track=_track(c), span=int(ts[-1]) + int(c["gap_us"]), turn=itertools.cycle(slots))


def _sizes(rng, lo, hi, n):
    return np.round(np.exp(rng.uniform(np.log(lo), np.log(hi), n))).astype(np.int64)


def _graph_sizes(c):
    """(|E|, changes each way) of every graph of a batched case: the same for every seed."""
    rng = np.random.default_rng(c["graphs"])
    ne = _sizes(rng, c["e_lo"], c["e_hi"], c["graphs"])
    return [(int(e), int(max(1, min(b, e) // 2))) for e, b in zip(ne, _sizes(rng, c["b_lo"], c["b_hi"], c["graphs"]))]


def _prepare_batched(c, seed):
    graphs = []
    for k, (ne, n) in enumerate(_graph_sizes(c)):
        one = dict(kind="batch", ne=ne, nv=max(c["hi"] * 4, ne // 2), alpha=2.5, lo=2, hi=c["hi"], s=0.0, q=0.0, changes=n,
                   track="hyperedge")
        graphs.append(_prepare_batch(one, seed * 1000 + k))
    return dict(kind="batched", graphs=graphs, launch=c["graph"])


def _tenant_sizes(c):
    rng = np.random.default_rng(c["tenants"])
    w = _sizes(rng, 1e4, 1e6, c["tenants"])
    ne = np.maximum(64, w * c["total"] // w.sum())
    return [(int(e), int(max(1, min(b, e) // 2))) for e, b in zip(ne, _sizes(rng, c["b_lo"], c["b_hi"], c["tenants"]))]


def _prepare_served(c, seed):
    server = hgt.Server(hbm_budget_bytes=8 << 30)
    tenants = []
    for k, (ne, n) in enumerate(_tenant_sizes(c)):
        one = dict(nv=max(64, ne // 2), alpha=2.0, lo=2, hi=c["hi"], s=1.3, q=c["q"])
        g, _, (off, mem) = _make_rows(one, seed * 1000 + k, ne + 2 * n)
        ts = _arrival_times(g, ne + 2 * n, 1000.0)
        o, m = _split(off, mem, 0, ne)
        t = server.add_tenant(one["nv"], o, m, ts[:ne].clone(), track=_track(dict(track=ALL)), window=600_000_000)
        dels = torch.randperm(ne, generator=g, device=DEV)[:n].cpu().numpy().astype(np.uint32)
        sets = []
        for j in range(2):
            o, m = _split(off, mem, ne + j * n, ne + (j + 1) * n)
            sets.append(dict(off=o.cpu().numpy().astype(np.uint64), mem=m.cpu().numpy().astype(np.uint32),
                             ts=ts[ne + j * n:ne + (j + 1) * n].cpu().numpy()))
        tenants.append(dict(t=t, ids=dels, turn=itertools.cycle(sets), span=int(ts[-1] - ts[ne]) + 1000))
    return dict(kind="served", server=server, tenants=tenants)


def _prepare_vertex_ops(c, seed):
    n = c["ops"]
    g, vert, (off, mem) = _make_rows(c, seed, c["ne"])
    h = torch.randperm(c["ne"], generator=g, device=DEV)
    low, length = off[h], off[h + 1] - off[h]
    # a member of each leaves, in the first half; a vertex that is no member of it enters, in the second
    pick = low + (torch.rand(len(h), generator=g, device=DEV) * length).long().clamp(max=length - 1)
    out = mem[pick]
    new = vert.draw(len(h)).to(torch.int32)
    row = torch.repeat_interleave(torch.arange(c["ne"], device=DEV), off[1:] - off[:-1])
    has = torch.zeros(c["ne"], dtype=torch.bool, device=DEV)
    by_edge = torch.empty(c["ne"], dtype=torch.int32, device=DEV)
    by_edge[h] = new
    has[row[by_edge[row] == mem]] = True
    fresh = h[n // 2:][~has[h[n // 2:]]][:n - n // 2]
    edges = torch.cat([h[:n // 2], fresh]).to(torch.int32)
    verts = torch.cat([out[:n // 2], by_edge[fresh]])
    insert = torch.zeros(len(edges), dtype=torch.uint8, device=DEV)
    insert[n // 2:] = 1
    order = torch.randperm(len(edges), generator=g, device=DEV)
    edges, verts, insert = edges[order].contiguous(), verts[order].contiguous(), insert[order].contiguous()
    graph = hgt.Graph.build(c["nv"], off, mem, track=_track(c))
    return dict(kind="vertex_ops", graph=graph, track=_track(c), edges=edges, verts=verts,
                turn=itertools.cycle([insert, 1 - insert]))


def prepare(case, seed):
    return {"batch": _prepare_batch, "dyadic": _prepare_batch, "stream": _prepare_stream, "batched": _prepare_batched,
            "served": _prepare_served, "vertex_ops": _prepare_vertex_ops}[case["kind"]](case, seed)


# --------------------------------------------------------------------------- #
# one pass
# --------------------------------------------------------------------------- #
def _counts(graph, track):
    return {k: np.array(graph.triad_counts(k), dtype=np.uint64) for k in track}


def run(state):
    kind = state["kind"]
    if kind == "batch":
        off, mem = next(state["turn"])
        state["ids"] = state["graph"].apply_batch(state["ids"], off, mem, noalloc=state["noalloc"])
        return dict(ids=state["ids"], counts=_counts(state["graph"], state["track"]))
    if kind == "stream":
        slot = next(state["turn"])
        slot["ts"] = slot["ts"] + state["span"]
        slot["ids"] = state["graph"].apply_batch(slot["ids"], slot["off"], slot["mem"], slot["ts"])
        return dict(ids=slot["ids"], counts=_counts(state["graph"], state["track"]))
    if kind == "vertex_ops":
        state["graph"].apply_vertex_ops(state["edges"], state["verts"], next(state["turn"]))
        return dict(counts=_counts(state["graph"], state["track"]))
    if kind == "batched":
        items = [(s["graph"], s["ids"], *next(s["turn"])) for s in state["graphs"]]
        ids = hgt.apply_batches(items, graph=state["launch"])
        for s, i in zip(state["graphs"], ids):
            s["ids"] = i
        return dict(ids=torch.cat(ids), counts=np.array([s["graph"].triad_counts("hyperedge") for s in state["graphs"]], dtype=np.uint64))
    server, tickets = state["server"], []
    for t in state["tenants"]:
        req = next(t["turn"])
        tickets.append(server.submit(t["t"], t["ids"], req["off"], req["mem"], req["ts"]))
        req["ts"] = req["ts"] + 2 * t["span"]  # stamps of this set's next turn
    done = [server.wait(k) for k in tickets]
    for t, d in zip(state["tenants"], done):
        t["ids"] = d["ids"]
    fam = ("hyperedge", "incident_vertex", "temporal")
    return dict(status=np.array([d["status"] for d in done]), ids=np.concatenate([d["ids"] for d in done]).astype(np.int64),
                counts={k: np.array([d[k] for d in done], dtype=np.uint64) for k in fam})


# --------------------------------------------------------------------------- #
# what a pass cannot do without
# --------------------------------------------------------------------------- #
def _one_batch(c, n_del, n_ins, temporal=False, share=1.0):
    """Bytes of one vertical batch, expected over the distributions: the batch itself,
    the incidence lists of the touched vertices once, the rows of the hyperedges on
    them once, and the changed rows and list entries written.  `share`: the part of
    a list that lies in the time window."""
    lo, hi = c.get("lo", 2), min(c.get("hi", 2), c["nv"] // 4)
    k = np.arange(lo, hi + 1, dtype=np.float64)
    w = k ** -c.get("alpha", 0.0)
    mean = float((k * w).sum() / w.sum())
    p = (np.arange(1, c["nv"] + 1, dtype=np.float64) + c["q"]) ** -c["s"]
    p /= p.sum()
    touched = -np.expm1(-(n_del + n_ins) * mean * p)          # a vertex is touched
    lists = float((touched * p).sum()) * c["ne"] * mean * share
    near = c["ne"] * share * -math.expm1(-mean * float((touched * p).sum()))
    entry = 12 if temporal else 4
    return (4 * n_del + 12 * n_ins + 4 * mean * n_ins + lists * entry + near * 4 * mean
            + (n_del + n_ins) * mean * (4 + entry))


def work(case):
    kind = case["kind"]
    if kind in ("batch", "dyadic"):
        b = _one_batch(case, case["changes"], case["changes"])
    elif kind == "stream":
        span = case["ne"] * case["gap_us"]
        share = min(1.0, (case["window_us"] + case["batch"] * case["gap_us"]) / span) if case["track"] == "temporal" else 1.0
        b = _one_batch(case, case["batch"], case["batch"], True, share)
    elif kind == "vertex_ops":
        b = 9 * case["ops"] + _one_batch(case, case["ops"], case["ops"])
    else:
        sizes = _graph_sizes(case) if kind == "batched" else _tenant_sizes(case)
        shape = dict(alpha=2.5, s=0.0, q=0.0) if kind == "batched" else dict(alpha=2.0, s=1.3, q=case["q"])
        b = sum(_one_batch(dict(nv=max(64, e // 2), ne=e, lo=2, hi=case["hi"], **shape), n, n, kind == "served") for e, n in sizes)
    return {"bytes": b, "flops": 0}


# --------------------------------------------------------------------------- #
# exact values: dense linear algebra and enumeration on small inputs
# --------------------------------------------------------------------------- #
def _codes():
    """Hyperedge classes: the Venn patterns of three connected sets up to relabelling,
    indexed by their smallest code (bits: a, b, c only; ab, bc, ca only; abc)."""
    bits = {(0,): 0, (1,): 1, (2,): 2, (0, 1): 3, (1, 2): 4, (0, 2): 5, (0, 1, 2): 6}
    best = {}
    for code in range(128):
        regions = [r for r, b in bits.items() if code >> b & 1]
        if not all(any(s in r for r in regions) for s in range(3)):
            continue
        if sum(any(x in r and y in r for r in regions) for x, y in ((0, 1), (1, 2), (0, 2))) < 2:
            continue
        best[code] = min(sum(1 << bits[tuple(sorted(p[s] for s in r))] for r in regions)
                         for p in itertools.permutations(range(3)))
    order = {k: i for i, k in enumerate(sorted(set(best.values())))}
    table = torch.full((128,), len(order), dtype=torch.int64)
    for code, k in best.items():
        table[code] = order[k]
    return table, len(order)


def exact(case, seed):
    """For a small vertical case: counts of the graph after its first batch."""
    if case["kind"] != "batch" or case["ne"] > 2_000 or case["nv"] > 5_000:
        return None  # enumeration would take minutes; the values are whole numbers
    (off, mem), dels, sets = _batch_inputs(case, seed)
    inc = torch.zeros(case["ne"], case["nv"], dtype=torch.float64)

    def fill(ids, o, m):
        inc[ids] = 0
        inc[torch.repeat_interleave(ids, (o[1:] - o[:-1]).cpu()), m.cpu().long()] = 1

    ids = dels.sort().values.cpu()
    fill(torch.arange(case["ne"]), off, mem)
    inc[ids.long()] = 0
    fill(ids.long(), *sets[0])
    inc = inc.to(DEV)
    track, counts = _track(case), {}
    if "hyperedge" in track:
        table, n = _codes()
        table, d = table.to(DEV), inc.sum(1).long()
        both = (inc @ inc.T).long()
        hist = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        for a in range(len(d) - 2):
            r = inc[a + 1:, inc[a] > 0]
            abc = (r @ r.T).long()
            ab, bc, db = both[a, a + 1:], both[a + 1:, a + 1:], d[a + 1:]
            x, y = ab[:, None], ab[None, :]
            code = ((d[a] - x - y + abc > 0).long() | (db[:, None] - x - bc + abc > 0).long() << 1
                    | (db[None, :] - y - bc + abc > 0).long() << 2 | (x - abc > 0).long() << 3
                    | (bc - abc > 0).long() << 4 | (y - abc > 0).long() << 5 | (abc > 0).long() << 6)
            hist += torch.bincount(table[code].triu(1).add(torch.ones_like(code).tril() * n).clamp(max=n).flatten(), minlength=n + 1)
        counts["hyperedge"] = hist[:n].cpu().numpy().astype(np.uint64)
    if "incident_vertex" in track:
        d = inc.sum(1)
        off_diag = 1 - torch.eye(case["nv"], dtype=torch.float64, device=DEV)
        m, w = (inc.T @ inc) * off_diag, (inc.T @ (inc * (d - 2)[:, None])) * off_diag
        t1 = int((d * (d - 1) * (d - 2) / 6).sum().round())
        t2 = int(((m * w).sum() / 2).round()) - 3 * t1
        every = int((((m @ m) * m).sum() / 6).round())
        counts["incident_vertex"] = np.array([t1, t2, every - t1 - t2], dtype=np.uint64)
    return dict(ids=ids.to(torch.int32), counts={k: counts[k] for k in track})
