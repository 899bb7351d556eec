"""Performance cases: what a program does with this library, from the smallest
call to the largest workload, through the public entry points of
paper_2507_20441_amd.timest.

Kinds of case (the "kind" of a case):
  edges   edge arrays on the device -> graph, then per motif the weights and
          the samples (a program that meets a new graph)
  query   one estimate on a resident graph (weights and samples)
  sample  samples from a resident weight set (more samples for a known motif)
  family  several motifs over one stream of tree samples
  batch   many (graph, motif) jobs in one call
  serve   a burst of queries at a running server whose sets are warm
  trees   choice of the spanning tree by its total weight

Graphs are the package's synthetic ones: power-law endpoints, bursty times.
"""
import math
from fractions import Fraction

import numpy as np
import torch

from paper_2507_20441_amd import timest as T
from paper_2507_20441_amd import workloads as W

ORDERED = tuple(W.MOTIFS)
# partial orders of the package, without the ones whose shape repeats
PARTIAL = ("po_fan3", "po_cycle3", "po_sg", "po_free2", "po_diamond")
# 4-vertex motifs that share the tree a->b->c->d
FAMILY_TREE = ((0, 1), (1, 2), (2, 3))
FAMILY = (((0, 1), (1, 2), (2, 3), (3, 0)), ((0, 1), (1, 2), (2, 3), (3, 1)), ((0, 1), (1, 2), (2, 0), (2, 3)),
          ((3, 0), (0, 1), (1, 2), (2, 3)))


def listed():
    graph_1m = dict(m=1_000_000, n=50_000, gamma=2.1, span=10_000_000, unit=1)
    return [
        # the smallest whole estimate: a graph of 20,000 edges, latency is what counts
        dict(name="tiny_from_edges", kind="edges", m=20_000, n=1_000, gamma=2.3, span=100_000, unit=1,
             times="uniform", motifs="3cycle", delta=1_000, k=100_000, keep=False),
        # a few more samples from a set that is there: the smallest call
        dict(name="small_sample_call", kind="sample", m=20_000, n=1_000, gamma=2.3, span=100_000, unit=1,
             times="uniform", motifs="3cycle", delta=1_000, k=9_973, records=False),
        # samples with their records, to look at single matches (odd count, several tree levels)
        dict(name="sample_records", kind="sample", m=200_003, n=5_000, gamma=2.1, span=3_000_000, unit=1,
             times="bursty", motifs="6chain", delta=3_600, k=150_001, records=True),
        # the medium workload: 2e6 edges, two motifs, 1e7 samples each
        dict(name="medium_from_edges", kind="edges", m=2_000_000, n=100_000, gamma=2.1, span=10_000_000, unit=1,
             times="bursty", motifs="4cycle,4star", delta=3_600, k=10_000_000, keep=True),
        # one query of an analyst on a resident graph: deep tree, a day's window
        dict(name="query_chain", kind="query", times="bursty", motifs="6chain", delta=86_400, k=1_000_003,
             constraints=3, **graph_1m),
        # timestamps in milliseconds (more than 32 bits of span)
        dict(name="query_milliseconds", kind="query", times="bursty", motifs="scatter_gather", delta=14_400,
             k=2_000_000, constraints=3, **dict(graph_1m, m=1_500_007, unit=1000)),
        # a motif whose edges are only partly ordered
        dict(name="query_partial_order", kind="query", times="bursty", motifs="po_sg", delta=3_600, k=300_000,
             constraints=3, m=200_000, n=5_000, gamma=2.1, span=3_000_000, unit=1),
        # all motifs on four vertices with the same tree, counted together
        dict(name="family", kind="family", times="bursty", delta=3_600, k=2_000_000, m=2_000_000, n=100_000,
             gamma=2.1, span=10_000_000, unit=1),
        # a queue of jobs over graphs of very different sizes
        dict(name="batch_jobs", kind="batch", jobs=16, m_lo=10_000, m_hi=1_000_000, k_lo=100_000, k_hi=2_000_000),
        # queries that reach a warm server together
        dict(name="serve_burst", kind="serve", graphs=2, m=1_000_000, n=50_000, gamma=2.1, span=10_000_000,
             queries=24, k_lo=100_000, k_hi=2_000_000),
        # which tree to sample from: three candidates weighed
        dict(name="choose_tree", kind="trees", times="bursty", motifs="scatter_gather", delta=3_600, candidates=3,
             m=2_000_000, n=100_000, gamma=2.1, span=10_000_000, unit=1),
        # the large workload: 1e8 edges, two motifs, 1e8 samples each
        dict(name="large_from_edges", kind="edges", m=100_000_000, n=2_000_000, gamma=2.0, span=30_000_000, unit=1,
             times="bursty", reciprocal=10_000_000, motifs="scatter_gather,6chain", delta=86_400, k=100_000_000,
             keep=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: up to 4e6 edges and 1e7 samples."""
    kind = rng.choice(("edges", "edges", "query", "query", "sample", "sample", "family", "batch", "serve", "trees"))
    if kind == "batch":
        return dict(kind=kind, jobs=rng.randint(2, 32), m_lo=10_000, m_hi=_log(rng, 50_000, 1_500_000),
                    k_lo=100_000, k_hi=_log(rng, 200_000, 3_000_000))
    if kind == "serve":
        m = _log(rng, 100_000, 1_500_000)
        return dict(kind=kind, graphs=rng.randint(1, 3), m=m, n=max(50, m // 20), gamma=2.1, span=10_000_000,
                    queries=rng.randint(4, 32), k_lo=100_000, k_hi=_log(rng, 200_000, 3_000_000))
    # the span follows the size, so that small graphs hold matches too
    m = _log(rng, 100_000 if kind == "trees" else 10_000, 4_000_000)
    case = dict(kind=kind, m=m, n=max(50, m // rng.randint(10, 40)), gamma=rng.choice((2.0, 2.1, 2.3)),
                span=max(300_000, m * rng.choice((2, 5, 15))), unit=rng.choice((1, 1, 1, 1000)),
                times="bursty", delta=_log(rng, 1_000, 86_400))
    if kind == "trees":
        return dict(case, motifs=rng.choice(ORDERED), candidates=rng.randint(2, 4))
    case["k"] = _log(rng, 5_000 if kind == "sample" else 100_000, 10_000_000)
    if kind == "family":
        return case
    if kind == "edges":
        return dict(case, motifs=rng.choice(ORDERED), keep=rng.random() < 0.5)
    if kind == "query":
        if rng.random() < 0.25:
            # partial orders: smaller windows and counts, as their completions are enumerated
            return dict(case, motifs=rng.choice(PARTIAL), delta=_log(rng, 1_000, 7_200),
                        k=_log(rng, 100_000, 1_000_000), constraints=3)
        return dict(case, motifs=rng.choice(ORDERED), constraints=rng.choice((3, 3, 3, 1)))
    records = rng.random() < 0.3
    if records:
        case["k"] = min(case["k"], 300_000)
    return dict(case, motifs=rng.choice(ORDERED), records=records)


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _edges(case, seed):
    """Device edge arrays of a case's graph."""
    if case.get("times", "bursty") == "uniform":
        g = W.chung_lu_graph(case["n"], case["m"], case["gamma"], seed, times="uniform", tmax=case["span"])
        u, v, t = (torch.from_numpy(x).cuda() for x in (g.src, g.dst, g.t))
    else:
        u, v, t = W.device_graph(case["n"], case["m"], case["gamma"], seed, span=case["span"],
                                 reciprocal=case.get("reciprocal", 0))
    if case.get("unit", 1) > 1:
        # finer clock: the second's fraction below it
        gen = torch.Generator(device=u.device)
        gen.manual_seed(seed)
        t = t * case["unit"] + torch.randint(0, case["unit"], t.shape, generator=gen, device=t.device)
    return u, v, t


def _motif(name, delta):
    if name in W.PO_MOTIFS:
        edges, before = W.PO_MOTIFS[name]
        return T.make_motif(edges, delta, before=before)
    return T.make_motif(W.MOTIFS[name], delta)


def _motifs(case):
    return [_motif(name, case["delta"] * case.get("unit", 1)) for name in case["motifs"].split(",")]


def _jobs(case, seed):
    """Jobs of the batched workload's ranges: sizes, motifs, windows, budgets."""
    rng = np.random.default_rng(seed)
    jobs = []
    for _ in range(case["jobs"]):
        m = int(round(math.exp(rng.uniform(math.log(case["m_lo"]), math.log(case["m_hi"])))))
        jobs.append(dict(m=m, n=max(50, m // 20), gamma=2.1, span=10_000_000, motif=ORDERED[rng.integers(len(ORDERED))],
                         delta=int(round(math.exp(rng.uniform(math.log(600), math.log(86_400))))),
                         k=int(round(math.exp(rng.uniform(math.log(case["k_lo"]), math.log(case["k_hi"]))))),
                         graph_seed=int(rng.integers(1 << 40)), seed=int(rng.integers(1, 1 << 62))))
    return jobs


def _queries(case, seed):
    rng = np.random.default_rng(seed)
    return [dict(graph=int(rng.integers(case["graphs"])), motif=ORDERED[rng.integers(len(ORDERED))],
                 delta=int(W.SERVE_DELTAS[rng.integers(len(W.SERVE_DELTAS))]),
                 k=int(round(math.exp(rng.uniform(math.log(case["k_lo"]), math.log(case["k_hi"]))))),
                 seed=int(rng.integers(1, 1 << 62))) for _ in range(case["queries"])]


def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case, seed=seed + 1)
    if kind == "edges":
        state["edges"] = _edges(case, seed)
        state["motifs"] = _motifs(case)
    elif kind in ("query", "trees"):
        state["graph"] = T.Graph(*_edges(case, seed), case["n"])
        state["motif"] = _motifs(case)[0]
    elif kind == "sample":
        state["weights"] = T.Weights(T.Graph(*_edges(case, seed), case["n"]), _motifs(case)[0])
    elif kind == "family":
        delta = case["delta"] * case.get("unit", 1)
        state["weights"] = T.Weights(T.Graph(*_edges(case, seed), case["n"]), T.make_motif(FAMILY_TREE, delta))
        state["motifs"] = [T.make_motif(e, delta) for e in FAMILY]
    elif kind == "batch":
        jobs = _jobs(case, seed)
        state["graphs"] = [T.Graph(*_edges(j, j["graph_seed"]), j["n"]) for j in jobs]
        state["motifs"] = [_motif(j["motif"], j["delta"]) for j in jobs]
        state["ks"] = [j["k"] for j in jobs]
        state["seeds"] = [j["seed"] for j in jobs]
    elif kind == "serve":
        server = T.Server(32 << 30)
        ids = [server.add_graph(T.Graph(*_edges(case, 1000 * seed + g), case["n"])) for g in range(case["graphs"])]
        queries = [dict(q, graph=ids[q["graph"]], motif=_motif(q["motif"], q["delta"])) for q in _queries(case, seed)]
        for ticket in [server.submit(q["graph"], q["motif"], 1000, 1) for q in queries]:
            server.wait(ticket)  # the sets are warm
        state["server"], state["queries"] = server, queries
    return state


# ---------------------------------------------------------------------------
# One pass.
# ---------------------------------------------------------------------------
def _out(r):
    """A result as its estimate, its standard error and every exact field."""
    return dict(estimate=r.estimate, std_error=r.std_error,
                sums=np.array([r.W.lo, r.W.hi, r.acc2.lo, r.acc2.hi, r.acc2_sq.lo, r.acc2_sq.hi, r.k, r.n_valid,
                               r.n_bad_vertex, r.n_bad_delta, r.n_bad_order, r.n_nonzero, r.q, r.flags],
                              np.uint64).view(np.int64))


def _outs(results):
    """The same of several results, row by row."""
    outs = [_out(r) for r in results]
    return dict(estimate=np.array([o["estimate"] for o in outs]), std_error=np.array([o["std_error"] for o in outs]),
                sums=np.stack([o["sums"] for o in outs]))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "edges":
        g = T.Graph(*state["edges"], case["n"])
        out = []
        for mo in state["motifs"]:
            if case["keep"]:
                w = T.Weights(g, mo)
                out.append(w.sample(state["seed"], case["k"])[0])
                w.close()
            else:
                out.append(T.estimate(g, mo, case["k"], state["seed"]))
        g.close()
        return _outs(out)
    if kind == "query":
        return _out(T.estimate(state["graph"], state["motif"], case["k"], state["seed"],
                               constraints=case["constraints"]))
    if kind == "sample":
        res, recs = state["weights"].sample(state["seed"], case["k"], records=case["records"])
        out = _out(res)
        if recs is not None:
            out["records"] = recs.view(np.int32).reshape(case["k"], -1)
        return out
    if kind == "family":
        return _outs(T.sample_family(state["weights"], state["motifs"], state["seed"], case["k"]))
    if kind == "batch":
        return _outs(T.estimate_batch(state["graphs"], state["motifs"], state["ks"], state["seeds"]))
    if kind == "serve":
        server = state["server"]
        tickets = [server.submit(q["graph"], q["motif"], q["k"], q["seed"]) for q in state["queries"]]
        return _outs([server.wait(t)[0] for t in tickets])
    tree, Ws = T.choose_tree(state["graph"], state["motif"], case["candidates"])
    return dict(weights=np.array([[w & (2**64 - 1), w >> 64] for w in Ws], np.uint64).view(np.int64),
                tree=np.array(list(tree.edge[:tree.n_edges]) + [tree.center], np.int64))


# ---------------------------------------------------------------------------
# What a pass cannot do without: every edge read once (ids and time, 16 bytes;
# 12 with the times in 32 bits), once more per weight set (its list entries:
# neighbour and time), a list entry per tree edge of every sample, and the
# records written.  Integer work: flops stay 0.
# ---------------------------------------------------------------------------
def _tree_edges(name):
    edges = W.PO_MOTIFS[name][0] if name in W.PO_MOTIFS else W.MOTIFS[name]
    return W.motif_vertices(edges) - 1


def work(case):
    kind = case["kind"]
    entry = 8 if case.get("unit", 1) == 1 else 12
    if kind == "batch":
        jobs = _jobs(case, 0)
        return {"bytes": sum(8 * j["m"] + 8 * j["k"] * _tree_edges(j["motif"]) for j in jobs), "flops": 0}
    if kind == "serve":
        return {"bytes": sum(8 * q["k"] * _tree_edges(q["motif"]) for q in _queries(case, 0)), "flops": 0}
    m = case["m"]
    if kind == "family":
        return {"bytes": len(FAMILY_TREE) * entry * case["k"], "flops": 0}
    if kind == "trees":
        return {"bytes": case["candidates"] * entry * m, "flops": 0}
    total = 16 * m if kind == "edges" else 0
    for name in case["motifs"].split(","):
        total += (entry * m if kind != "sample" else 0) + entry * case["k"] * _tree_edges(name)
    if case.get("records"):
        total += 64 * case["k"]
    return {"bytes": total, "flops": 0}


# ---------------------------------------------------------------------------
# The same outputs in plain numpy and Python integers, from the definitions
# (Alg. 1-6 of the paper, totally ordered motifs): candidate lists, weights
# and inverse-CDF picks edge by edge and sample by sample.
# ---------------------------------------------------------------------------
TREES = {"3cycle": ((0, 1), 0), "4cycle": ((0, 1, 2), 1), "4star": ((0, 1, 2, 3), 0),
         "scatter_gather": ((0, 1, 4, 5), 1), "6chain": ((0, 1, 2, 3, 4), 2)}


def _philox(seed, k, d):
    """Philox4x32-10 blocks of draw d of samples 0 .. k-1, as Python integers."""
    lo32 = np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)
    j = np.arange(k, dtype=np.uint64)
    c = [j & lo32, j >> s32, np.full(k, d, np.uint64), np.zeros(k, np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> s32) ^ c[1] ^ np.uint64(k0), p1 & lo32, (p0 >> s32) ^ c[3] ^ np.uint64(k1), p0 & lo32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    lo, hi = c[0] | (c[1] << s32), c[2] | (c[3] << s32)
    return [(int(h) << 64) | int(x) for h, x in zip(hi, lo)]


class _Exact:
    def __init__(self, u, v, t, edges, tree, center, delta):
        order = np.lexsort((v, u, t))
        self.u, self.v = u[order].astype(np.int64), v[order].astype(np.int64)
        self.t = t[order] - t.min()
        self.m, self.edges, self.delta = len(u), edges, delta
        self.q = int(self.t[-1]) // delta + 1
        # per vertex: eids, times and neighbours of its out- and in-list in eid order
        self.lists = []
        for own, nbr in ((self.u, self.v), (self.v, self.u)):
            by = np.argsort(own, kind="stable")
            cut = np.flatnonzero(np.diff(own[by])) + 1
            self.lists.append({int(own[x[0]]): (x, self.t[x], nbr[x]) for x in np.split(by, cut)})
        # pairs (x, y) -> sorted times
        key = self.u * (max(self.u.max(), self.v.max()) + 1) + self.v
        by = np.argsort(key, kind="stable")
        self.pair = {(int(self.u[x[0]]), int(self.v[x[0]])): self.t[x]
                     for x in np.split(by, np.flatnonzero(np.diff(key[by])) + 1)}
        # pre-order: the center, then children by increasing index
        self.slots, rest = [], set(tree) - {center}

        # children are fixed before any subtree is entered
        def claim(e, parent, at):
            s = len(self.slots)
            self.slots.append(dict(e=e, parent=parent, at=at, kids=[]))
            if parent >= 0:
                self.slots[parent]["kids"].append(s)
            mine = [(c, [x for x in edges[e] if x in edges[c] and x != at][0]) for c in sorted(rest)
                    if any(x in edges[c] and x != at for x in edges[e])]
            for c, _ in mine:
                rest.discard(c)
            for c, x in mine:
                claim(c, s, x)

        claim(center, -1, None)
        self._weights()

    def window(self, s, e, i):
        """Candidate eids of slot s for its parent matched to eid e in interval i."""
        sl = self.slots[s]
        pe = self.edges[self.slots[sl["parent"]]["e"]]
        ends = (int(self.u[e]), int(self.v[e]))
        g, o = ends if pe[0] == sl["at"] else ends[::-1]
        entry = self.lists[0 if self.edges[sl["e"]][0] == sl["at"] else 1].get(g)
        if entry is None:
            return np.zeros(0, np.int64)
        te = int(self.t[e])
        if sl["e"] < self.slots[sl["parent"]]["e"]:
            lo, hi = max(te - self.delta, i * self.delta), te
        else:
            lo, hi = te, min(te + self.delta, (i + 2) * self.delta - 1)
        eids, times, nbr = entry
        a, b = np.searchsorted(times, lo, "left"), np.searchsorted(times, hi, "right")
        return eids[a:b][nbr[a:b] != o]

    def _weights(self):
        blk = (self.t // self.delta).tolist()
        self.w = {}
        for s in reversed(range(len(self.slots))):
            kids = self.slots[s]["kids"]
            if not kids and s:
                continue
            w = np.zeros((2, self.m), np.int64)
            for e, b in enumerate(blk):
                for i in ((b, b - 1) if b else (b,)):
                    p = 1
                    for c in kids:
                        cand = self.window(c, e, i)
                        p *= int(self.w[c][i & 1][cand].sum()) if self.slots[c]["kids"] else len(cand)
                    w[i & 1, e] = p
            self.w[s] = w
        lo = np.searchsorted(self.t, np.arange(self.q) * self.delta, "left")
        hi = np.searchsorted(self.t, (np.arange(self.q) + 2) * self.delta, "left")
        self.pi = np.repeat(np.arange(self.q), hi - lo)
        self.pe = np.concatenate([np.arange(a, b) for a, b in zip(lo, hi)])
        self.cum = np.cumsum(self.w[0][self.pi & 1, self.pe])
        self.W = int(self.cum[-1])

    def completions(self, img, times):
        """Assignments of the non-tree edges, strictly increasing and within delta."""
        total, l, p = 1, len(self.edges), 0
        first, last = min(times.values()), max(times.values())
        while p < l:
            if p in times:
                p += 1
                continue
            r = p
            while r < l and r not in times:
                r += 1
            lo = times[p - 1] + 1 if p else last - self.delta
            hi = times[r] - 1 if r < l else first + self.delta
            chains = None  # per entry of the run's last list: chains that end there
            for f in range(p, r):
                x = self.pair.get((img[self.edges[f][0]], img[self.edges[f][1]]), np.zeros(0, np.int64))
                x = x[np.searchsorted(x, lo, "left"):np.searchsorted(x, hi, "right")]
                if chains is None:
                    chains = (x, np.ones(len(x), np.int64))
                else:
                    before = np.concatenate(([0], np.cumsum(chains[1])))
                    chains = (x, before[np.searchsorted(chains[0], x, "left")])
            total *= int(chains[1].sum())
            p = r
        return total

    def sample(self, seed, k):
        nt = len(self.slots)
        X = [_philox(seed, k, d) for d in range(nt)]
        rank = {e: x for x, e in enumerate(sorted(sl["e"] for sl in self.slots))}
        rec = np.zeros(k, T.REC_DTYPE)
        rec["eid"] = -1
        rows = np.searchsorted(self.cum, np.array([(x * self.W) >> 128 for x in X[0]], np.int64), "right")
        s1 = s2 = 0
        count = [0, 0, 0, 0]
        nonzero = 0
        for j in range(k):
            i = int(self.pi[rows[j]])
            eid = [int(self.pe[rows[j]])]
            for s in range(1, nt):
                cand = self.window(s, eid[self.slots[s]["parent"]], i)
                if self.slots[s]["kids"]:
                    c = np.cumsum(self.w[s][i & 1][cand])
                    eid.append(int(cand[np.searchsorted(c, (X[s][j] * int(c[-1])) >> 128, "right")]))
                else:
                    eid.append(int(cand[(X[s][j] * len(cand)) >> 128]))
            img, times = {}, {}
            for sl, e in zip(self.slots, eid):
                a, b = self.edges[sl["e"]]
                img[a], img[b] = int(self.u[e]), int(self.v[e])
                times[sl["e"]] = int(self.t[e])
                rec["eid"][j, rank[sl["e"]]] = e
            ts = [times[e] for e in sorted(times)]
            status = n_phi = m_phi = 0
            if len(set(img.values())) < len(img):
                status = 1
            elif max(ts) - min(ts) > self.delta:
                status = 2
            elif any(x >= y for x, y in zip(ts, ts[1:])):
                status = 3
            else:
                b = ts[0] // self.delta
                n_phi = (1 if b < self.q else 0) + (1 if b and ts[-1] < (b + 1) * self.delta else 0)
                m_phi = self.completions(img, times)
                term = m_phi * (2 // n_phi)
                s1, s2 = s1 + term, s2 + term * term
                nonzero += m_phi > 0
            count[status] += 1
            rec["interval"][j], rec["status"][j], rec["n_phi"][j] = i, status, n_phi
            rec["m_lo"][j] = m_phi
        est = float(Fraction(self.W) * Fraction(s1, 2 * k))
        se = self.W / 2 * math.sqrt(Fraction(k * s2 - s1 * s1, k * k * (k - 1)))
        sums = [self.W, 0, s1, 0, s2, 0, k] + count + [nonzero, self.q, 0]
        return dict(estimate=est, std_error=se, sums=np.array(sums, np.int64)), rec


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("edges", "query", "sample") or case["motifs"] not in TREES or case.get("constraints", 3) != 3:
        return None
    nt = len(TREES[case["motifs"]][0])
    # about 15 us per window of an edge or a sample
    if 15e-6 * (2 * case["m"] * (nt - 1) + case["k"] * (nt + 1)) > 18:
        return None
    tree, center = TREES[case["motifs"]]
    u, v, t = (x.cpu().numpy() for x in _edges(case, seed))
    ref = _Exact(u, v, t.astype(np.int64), W.MOTIFS[case["motifs"]], tree, center,
                 case["delta"] * case.get("unit", 1))
    if not 0 < ref.W < 1 << 62:
        return None
    out, rec = ref.sample(seed + 1, case["k"])
    if kind == "sample":
        if case["records"]:
            out["records"] = rec.view(np.int32).reshape(case["k"], -1)
        return out
    if kind == "edges":
        return {name: np.array([value]) for name, value in out.items()}
    return out
