"""The framework's work as measured cases.

Every case goes through the package's public entry points on graphs of the
repository's own sizes:

  tiny     10 000 vertices,    16 predicates (Zipf 1.1),     100 000 triples
  medium   2 000 000 vertices, 64 predicates (Zipf 1.1),  20 000 000 triples
  large   40 000 000 vertices, 1024 predicates (Zipf 1.2), 200 000 000 triples

A graph is loaded and indexed once per process, as a program that answers
queries over it does; what the seed of a case picks are the queries (from a
log of chains, stars and snowflakes whose result sizes are known exactly) or,
for `load_build`, the triples.  Out-degrees follow a power law of exponent
2.2, objects are hubs or (three in ten) near their subject, so that cycles
close.

Kinds:
  single   a client that sends one BGP after another and reads every answer
           (`evaluate`: plan, join, fetch to the host)
  cyclic   the same with triangles and squares: large intermediate tables, a
           membership filter, few answers
  star     the same with star centres bound from patterns with constants (the
           intersection of sorted lists), in the static plan mode
  noalloc  a prepared program inside a tight loop: plans kept, answers left in
           the caller's device buffers
  count    an analytic query over the large graph: the answer stays on the
           device, the program reads its size, the steps' row counts and one
           page of 1000 rows
  fetch    a query with an OFFSET and a LIMIT of up to millions of rows, read to the
           host
  ext      OPTIONAL and FILTER queries, every answer read
  batch    the requests of many clients answered together, every answer read
  sweep    thousands of BGPs answered together on the large graph: the sizes
           of all answers are read, and some answers whole
  serve    the request loop: plans submitted, stepped and polled, every answer
           read
  load_build  triples loaded from host arrays and indexed; statistics of every
           predicate, the first page of the largest predicate's pairs and the
           subjects of the largest hub
"""
import math

import numpy as np
import torch

import paper_1807_07691_amd as G

GRAPHS = {
    "tiny": {"V": 10_000, "P": 16, "T": 100_000, "zipf": 1.1, "cap": 2_000, "templates": 240,
             "dense_div": 0},
    "medium": {"V": 2_000_000, "P": 64, "T": 20_000_000, "zipf": 1.1, "cap": 2_000,
               "templates": 600, "dense_div": 0},
    # more dense row pointers than the default, as the repository's benchmark has
    "large": {"V": 40_000_000, "P": 1_024, "T": 200_000_000, "zipf": 1.2, "cap": 100_000,
              "templates": 300, "dense_div": 256},
}
GRAPH_SEED = 7
_MANY = 10 ** 11  # counts saturate here, so that sums of a predicate's pairs stay exact
MODES = {"default": G.PLAN_DEFAULT, "adaptive": G.PLAN_ADAPTIVE}


def listed():
    return [
        # the smallest calls: one or two patterns around a constant, up to 100 rows each
        {"name": "point_lookups", "kind": "single", "graph": "medium", "queries": 16,
         "pats_lo": 1, "pats_hi": 2, "rows_lo": 1, "rows_hi": 100, "mode": "adaptive"},
        # ordinary interactive queries
        {"name": "interactive", "kind": "single", "graph": "medium", "queries": 16,
         "pats_lo": 3, "pats_hi": 5, "rows_lo": 300, "rows_hi": 30_000, "mode": "adaptive"},
        # an export: millions of rows to the host
        {"name": "export_rows", "kind": "fetch", "graph": "medium", "queries": 1,
         "pats_lo": 3, "pats_hi": 3, "rows_lo": 3_000_000, "rows_hi": 9_000_000,
         "mode": "adaptive"},
        # triangles: graph pattern matching with a closing edge
        {"name": "triangles", "kind": "cyclic", "graph": "medium", "queries": 4, "nodes": 3,
         "paths_lo": 1_000_000, "paths_hi": 30_000_000, "mode": "adaptive"},
        # entities that satisfy several constant conditions
        {"name": "star_conditions", "kind": "star", "graph": "large", "queries": 16,
         "members": 2, "hub_rank": 16, "mode": "default"},
        # prepared queries in a loop that may not allocate
        {"name": "prepared_loop", "kind": "noalloc", "graph": "medium", "queries": 16,
         "pats_lo": 2, "pats_hi": 4, "rows_lo": 1_000, "rows_hi": 100_000, "mode": "adaptive"},
        # the largest single answers
        {"name": "analytic_count", "kind": "count", "graph": "large", "queries": 2,
         "pats_lo": 2, "pats_hi": 5, "rows_lo": 50_000_000, "rows_hi": 400_000_000,
         "mode": "adaptive"},
        {"name": "optional_filter", "kind": "ext", "graph": "medium", "queries": 8,
         "pats_lo": 2, "pats_hi": 4, "rows_lo": 1_000, "rows_hi": 100_000, "mode": "adaptive"},
        # a web service's batch window
        {"name": "batch_60", "kind": "batch", "graph": "medium", "queries": 60,
         "pats_lo": 1, "pats_hi": 6, "rows_lo": 1, "rows_hi": 30_000, "mode": "adaptive"},
        # the benchmark's workload: result sizes spread over the decades of [1, 10^6]
        {"name": "sweep_4096", "kind": "sweep", "graph": "large", "queries": 4096,
         "pats_lo": 1, "pats_hi": 6, "rows_lo": 1, "rows_hi": 1_000_000, "mode": "adaptive"},
        {"name": "served_60", "kind": "serve", "graph": "medium", "queries": 60,
         "pats_lo": 1, "pats_hi": 5, "rows_lo": 1, "rows_hi": 30_000, "mode": "adaptive"},
        # a new data set: load, index, first answer
        {"name": "load_build_20m", "kind": "load_build", "triples": 20_000_000,
         "vertices": 2_000_000, "predicates": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "fetch", "cyclic", "star", "noalloc", "count", "ext",
                       "batch", "sweep", "serve", "load_build"])
    if kind == "load_build":
        t = _log(rng, 20_000, 20_000_000)
        return {"kind": kind, "triples": t, "vertices": max(64, int(t / rng.uniform(3, 20))),
                "predicates": rng.randint(1, 200)}
    graph = rng.choice(["tiny", "medium", "medium"])
    if kind == "star":
        return {"kind": kind, "graph": rng.choice(["medium", "large"]),
                "queries": rng.randint(3, 24), "members": rng.randint(2, 4),
                "hub_rank": _log(rng, 4, 100), "mode": rng.choice(["default", "adaptive"])}
    if kind == "cyclic":
        # wide enough that the graph has predicates with such path counts
        lo = _log(rng, 2_000, 20_000) if graph == "tiny" else _log(rng, 100_000, 5_000_000)
        return {"kind": kind, "graph": graph, "queries": rng.randint(1, 5),
                "nodes": rng.choice([3, 3, 4]), "paths_lo": lo, "paths_hi": lo * 12,
                "mode": "adaptive"}
    if kind == "sweep":
        return {"kind": kind, "graph": rng.choice(["medium", "large"]),
                "queries": _log(rng, 100, 4096), "pats_lo": 1, "pats_hi": rng.randint(4, 6),
                "rows_lo": 1, "rows_hi": _log(rng, 10_000, 1_000_000), "mode": "adaptive"}
    if kind == "count":
        lo = _log(rng, 2_000_000, 60_000_000)
        return {"kind": kind, "graph": "large", "queries": rng.randint(1, 3), "pats_lo": 2,
                "pats_hi": 5, "rows_lo": lo, "rows_hi": lo * 6, "mode": "adaptive"}
    if kind == "fetch":
        lo = _log(rng, 100_000, 2_000_000)
        n = rng.randint(1, 5)
        return {"kind": kind, "graph": "medium", "queries": 1, "pats_lo": n,
                "pats_hi": n, "rows_lo": lo, "rows_hi": lo * 4, "mode": "adaptive"}
    lo = _log(rng, 1, 10_000 if graph == "medium" else 500)
    q = {"kind": kind, "graph": graph, "queries": rng.randint(4, 60), "pats_lo": 1,
         "pats_hi": rng.randint(3, 6), "rows_lo": lo, "rows_hi": lo * rng.randint(10, 40),
         "mode": "adaptive"}
    if kind == "ext":
        q.update(queries=rng.randint(2, 12), pats_lo=2, mode="adaptive")
    if kind in ("single", "noalloc"):
        q["queries"] = rng.randint(4, 24)
    if kind == "noalloc":
        q["rows_hi"] = min(q["rows_hi"], 100_000)
    return q


# ---------------------------------------------------------------- graphs

def _triples(V, P, T, zipf, cap, seed):
    """(s, p, o) int32 device tensors: T triples, a few of them repeated."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dev = "cuda"
    deg = torch.rand(V, generator=g, device=dev, dtype=torch.float64).clamp_min_(1e-12)
    cdf = deg.pow_(-1 / 1.2).floor_().clamp_(max=cap).cumsum_(0)
    s = torch.empty(T, dtype=torch.int32, device=dev)
    p = torch.empty(T, dtype=torch.int32, device=dev)
    o = torch.empty(T, dtype=torch.int32, device=dev)
    w = torch.arange(1, P + 1, device=dev, dtype=torch.float64).pow_(-zipf).cumsum_(0)
    mult, add = 1_000_003, 12_345  # a bijection of the ids: no size is a multiple of 1 000 003
    step = 1 << 25
    for a in range(0, T, step):
        n = min(step, T - a)

        def uni():
            return torch.rand(n, generator=g, device=dev, dtype=torch.float64)

        si = torch.searchsorted(cdf, uni() * cdf[-1]).clamp_(max=V - 1)
        hub = (uni().pow_(3) * V).long().clamp_(max=V - 1) * mult % V
        near = (si + 1 + (-uni().clamp_min_(1e-12).log_() * 16).long()) % V
        s[a:a + n] = (si * mult + add) % V
        o[a:a + n] = (torch.where(uni() < 0.3, near, (hub + 7) % V) * mult + add) % V
        p[a:a + n] = torch.searchsorted(w, uni() * w[-1]).clamp_(max=P - 1)
    return s, p, o


class _Graph:
    """A loaded graph, its query log (exact result sizes) and its hubs."""

    def __init__(self, name):
        c = GRAPHS[name]
        self.V, self.P = c["V"], c["P"]
        s, p, o = _triples(c["V"], c["P"], c["T"], c["zipf"], c["cap"], GRAPH_SEED)
        self.store = G.gsmat_load_triples(s.cpu().numpy(), p.cpu().numpy(), o.cpu().numpy(),
                                          c["V"], c["P"])
        G.gsmat_build_index(self.store, c["dense_div"])
        # distinct triples by predicate and by either end, for the exact counts
        s, p, o = s.long(), p.long(), o.long()
        V = c["V"]
        key = ((p * V + s) * V + o).sort().values
        key = torch.unique_consecutive(key)
        self.by = [self._rows(key, V)]
        key = ((key // V // V * V + key % V) * V + key // V % V).sort().values
        self.by.append(self._rows(key, V))
        del s, p, o, key
        self.rng = np.random.default_rng(GRAPH_SEED)
        self.weight = np.arange(1, c["P"] + 1) ** -(0.7 * c["zipf"])
        self.weight /= self.weight.sum()
        self.log = []
        for _ in range(c["templates"]):
            self._template()
        self.size = np.array([q[1] for q in self.log], np.float64)
        self.pats = np.array([len(q[0]) for q in self.log])
        self.free = np.array([q[2] for q in self.log])
        self.paths = self._path_counts() if name != "large" else None
        self.hubs = self._hubs()
        del self.by
        torch.cuda.empty_cache()

    def _rows(self, key, V):
        """Sorted (predicate, vertex, neighbour) keys as rows: per predicate its
        vertices, their first positions and all neighbours."""
        row = key // V
        first = torch.ones_like(row, dtype=torch.bool)
        first[1:] = row[1:] != row[:-1]
        at = first.nonzero()[:, 0]
        row = row[at]
        bounds = torch.arange(self.P + 1, device="cuda") * V
        return {"vertex": row % V, "at": at, "nbr": (key % V).int(),
                "row0": torch.searchsorted(row, bounds).tolist(),
                "key0": torch.searchsorted(key, bounds * V).tolist()}

    def _message(self, p, out, w):
        """Per vertex: the sum of w over its neighbours along p (w None: ones)."""
        b = self.by[0 if out else 1]
        r0, r1, k0, k1 = b["row0"][p], b["row0"][p + 1], b["key0"][p], b["key0"][p + 1]
        got = torch.zeros(self.V, device="cuda", dtype=torch.int64)
        if r1 > r0:
            at = b["at"][r0:r1] - k0
            end = torch.cat([at[1:], at.new_tensor([k1 - k0])])
            if w is not None:
                run = torch.zeros(k1 - k0 + 1, device="cuda", dtype=torch.int64)
                torch.cumsum(w[b["nbr"][k0:k1].long()], 0, out=run[1:])
                at, end = run[at], run[end]
            got[b["vertex"][r0:r1]] = (end - at).clamp_(max=_MANY)
        return got

    def _template(self):
        """One query shape: a tree of 1-6 patterns; the log receives it with all
        its nodes free, and with constants at its first leaf, where its tables
        on the way stay within 20 times its answer (or a few thousand rows)."""
        r = self.rng
        n = int(r.integers(1, 7))
        shape = r.choice(["chain", "sstar", "ostar", "snow"])
        edges = []  # (parent, child, predicate, parent is the subject); node 0 is a leaf
        for c in range(1, n + 1):
            if shape == "chain":
                par, out = c - 1, bool(r.integers(0, 5))
            elif shape == "ostar":
                par, out = min(c - 1, 1), c == 1
            elif shape == "sstar" or c <= (n + 1) // 2 + 1:
                par, out = min(c - 1, 1), c > 1
            else:
                par, out = int(r.integers(2, c)), True
            edges.append((par, c, int(r.choice(self.P, p=self.weight)), out))
        w = self._count(edges)
        most = w  # rows of the largest part of the shape, joined in its order
        for k in range(1, n):
            most = torch.maximum(most, self._count(edges[:k]))
        total, top = float(w.sum(dtype=torch.float64)), float(most.sum(dtype=torch.float64))
        if total >= 1 and top <= max(20 * total, 100_000):
            self.log.append((self._pats(edges, None), total, True))
        some = ((w > 0) & (most <= (20 * w).clamp_(min=10_000))).nonzero()[:, 0]
        if len(some):
            some = some[torch.from_numpy(r.integers(0, len(some), 20_000)).cuda()]
            rows = w[some].cpu().numpy()
            some = some.cpu().numpy()
            for lo in 10 ** np.arange(7):
                idx = np.nonzero((rows >= lo) & (rows < lo * 10))[0]
                if len(idx):
                    for i in r.choice(idx, 8):
                        self.log.append((self._pats(edges, int(some[i])), float(rows[i]), False))

    def _count(self, edges):
        """Rows of the tree of patterns for each value of node 0."""
        w = {}
        for par, c, p, out in reversed(edges):
            m = self._message(p, out, w.pop(c, None))
            w[par] = m if par not in w else (w[par].double() * m).clamp_(max=_MANY).long()
        return w[0]

    @staticmethod
    def _pats(edges, root):
        def term(x):
            if x == 0 and root is not None:
                return root
            return -(x + 1) if root is None else -x
        return np.array([[term(a), p, term(b)] if out else [term(b), p, term(a)]
                         for a, b, p, out in edges], np.int32)

    def _path_counts(self):
        """Rows of (x p y, y q z) for the frequent predicates."""
        n = min(self.P, 24)
        ins = torch.stack([self._message(p, False, None).double() for p in range(n)])
        outs = torch.stack([self._message(p, True, None).double() for p in range(n)])
        return (ins @ outs.t()).cpu().numpy()

    def _hubs(self):
        """Objects with many subjects, per frequent predicate."""
        return [self._message(p, False, None).topk(512).indices.cpu().numpy()
                for p in range(min(self.P, 8))]

    def pick(self, case, r):
        """Queries of the log in the case's ranges, spread over the decades."""
        lo, hi = case["rows_lo"], case["rows_hi"]
        ok = ((self.pats >= case["pats_lo"]) & (self.pats <= case["pats_hi"]) &
              (self.size >= lo) & (self.size < hi))
        if case["kind"] == "count":
            ok &= self.free
        if case["kind"] == "noalloc":  # its tables have to fit 64 MiB
            ok &= ~self.free
        idx = np.nonzero(ok)[0]
        if case["kind"] == "fetch":  # at least the limit, and no more than the card holds
            idx = np.nonzero(self.free & (self.pats == case["pats_lo"]) &
                             (self.size >= lo) & (self.size < 40 * hi))[0]
            idx = idx[np.argsort(self.size[idx], kind="stable")[:12]]
        if len(idx) == 0:  # no query of that size: the nearest ones
            near = np.abs(np.log(self.size / math.sqrt(lo * hi)))
            near[self.size >= hi] += 50
            near[self.pats < case["pats_lo"]] += 100
            if case["kind"] == "count":
                near[~self.free | (self.size > 1e9)] += 200
            if case["kind"] == "noalloc":
                near[self.free] += 200
            idx = np.argsort(near, kind="stable")[:8]
        dec = np.floor(np.log10(self.size[idx])).astype(int)
        bins = [r.permutation(idx[dec == d]) for d in np.unique(dec)]
        got, at = [], 0
        while len(got) < case["queries"]:
            b = bins[at % len(bins)]
            got.append(int(b[(at // len(bins)) % len(b)]))
            at += 1
        return [self.log[i] for i in r.permutation(got)]

    def cycles(self, case, r):
        """Triangles (x p y, y q z, x t z) or squares whose two-step paths
        number as the case says."""
        ij = np.argwhere((self.paths >= case["paths_lo"]) & (self.paths <= case["paths_hi"]))
        if len(ij) == 0:
            d = np.abs(np.log(self.paths.clip(1) / math.sqrt(case["paths_lo"] * case["paths_hi"])))
            ij = np.stack(np.unravel_index(np.argsort(d, axis=None)[:8], d.shape), 1)
        out = []
        for _ in range(case["queries"]):
            a, b = (int(x) for x in ij[r.integers(0, len(ij))])
            t = int(r.integers(0, 6))
            if case["nodes"] == 3:
                out.append(np.array([[-1, a, -2], [-2, b, -3], [-1, t, -3]], np.int32))
            else:
                u = int(r.integers(8, 16))
                out.append(np.array([[-1, a, -2], [-2, b, -3], [-3, u, -4], [-1, t, -4]],
                                    np.int32))
        return out

    def stars(self, case, r):
        """A centre with constant objects on `members` patterns and one free leaf."""
        out = []
        for _ in range(case["queries"]):
            ps = r.choice(len(self.hubs), case["members"], replace=False)
            q = [[-1, int(p), int(self.hubs[p][r.integers(0, case["hub_rank"])])] for p in ps]
            q.append([-1, int(r.integers(0, min(self.P, 8))), -2])
            out.append(np.array(q, np.int32))
        return out


_graphs = {}


def _graph(name):
    if name not in _graphs:
        _graphs[name] = _Graph(name)
    return _graphs[name]


# ---------------------------------------------------------------- cases

def prepare(case, seed):
    r = np.random.default_rng([seed, 11])
    kind = case["kind"]
    if kind == "load_build":
        s, p, o = _triples(case["vertices"], case["predicates"], case["triples"], 1.1, 2_000,
                           seed)
        hub = int(torch.bincount(o).argmax())
        return {"kind": kind, "s": s.cpu().numpy(), "p": p.cpu().numpy(), "o": o.cpu().numpy(),
                "V": case["vertices"], "P": case["predicates"], "limit": case["triples"] // 20,
                "scan": np.array([[-1, 0, -2]], np.int32),
                "hub": np.array([[-1, 0, hub]], np.int32),
                "buf": np.zeros(case["triples"] // 8, np.int32)}
    g = _graph(case["graph"])
    mode = MODES[case["mode"]]
    st = {"kind": kind, "store": g.store, "mode": mode}
    if kind == "cyclic":
        st["queries"] = g.cycles(case, r)
    elif kind == "star":
        st["queries"] = g.stars(case, r)
    else:
        picked = g.pick(case, r)
        st["queries"] = [q[0] for q in picked]
    if kind == "noalloc":
        st["plans"] = [G.gsmat_plan(g.store, q, mode) for q in st["queries"]]
        st["out"] = torch.full((len(st["plans"]), case["pats_hi"] + 1, case["rows_hi"]), -1,
                               dtype=torch.int32, device="cuda")
    elif kind == "count":
        st["buf"] = np.zeros(case["queries"] * 1000 * (case["pats_hi"] + 1), np.int32)
    elif kind == "sweep":
        st["buf"] = np.zeros(8 * 30_000 * (case["pats_hi"] + 1), np.int32)
    elif kind in ("cyclic", "star"):
        st["buf"] = np.zeros(4_000_000, np.int32)
    elif kind == "fetch":
        st["limit"] = case["rows_lo"]
        st["offset"] = int(r.integers(0, max(1, int(picked[0][1]) - case["rows_lo"])))
    else:  # where the client gathers the answers
        st["buf"] = np.zeros(case["queries"] * case["rows_hi"] * (case["pats_hi"] + 2), np.int32)
    if kind == "ext":
        st["queries"] = [_optional(q, g.P, r) for q in st["queries"]]
    if kind == "sweep":
        # answers read whole: eight, from the smallest to 30 000 rows
        z = np.array([q[1] for q in picked])
        order = np.argsort(z, kind="stable")
        order = order[z[order] <= 30_000]
        st["read"] = [int(order[i]) for i in np.linspace(0, len(order) - 1, 8).astype(int)]
        st["packed"] = G.pack_queries(st["queries"])
    if kind == "serve":
        st["server"] = G.gsmat_server_new(g.store, mem_budget_bytes=32 << 30,
                                          max_active=len(st["queries"]))
    return st


def _optional(q, P, r):
    """The BGP as the required group, an OPTIONAL neighbour of its last
    variable along a frequent predicate, and FILTER (?v0 != ?v1)."""
    nv = int(-q[:, [0, 2]].min())
    pats = np.concatenate([q, np.zeros((len(q), 2), np.int32)], 1).tolist()
    pats.append([-nv, int(r.integers(0, min(P, 8))), -(nv + 1), 0, 1])
    return (np.array(pats, np.int32), np.array([[G.F_NE, -1, -2, 0]], np.int32), nv + 1)


def _gather(buf, answers):
    """The answers' sizes, and their rows one after the other in the client's
    buffer (up to its end)."""
    rows, at = np.zeros(len(answers), np.int64), 0
    for i, a in enumerate(answers):
        rows[i] = len(a)
        m = min(a.size, buf.size - at)
        buf[at:at + m] = a.ravel()[:m]
        at += m
    return [rows, buf]


def run(state):
    kind = state["kind"]
    if kind == "load_build":
        st = G.gsmat_load_triples(state["s"], state["p"], state["o"], state["V"], state["P"])
        G.gsmat_build_index(st)
        stats = np.array([G.gsmat_pred_stats(st, i) for i in range(state["P"])], np.int64)
        pl = G.gsmat_plan(st, state["scan"])
        res = G.gsmat_join(st, pl)
        page = G.gsmat_fetch_bindings(res, 0, state["limit"])
        hub = G.evaluate(st, state["hub"])
        res.close()
        pl.close()
        st.close()
        return [stats, page] + _gather(state["buf"], [hub])
    store, mode, queries = state["store"], state["mode"], state["queries"]
    if kind in ("single", "cyclic", "star"):
        return _gather(state["buf"], [G.evaluate(store, q, mode) for q in queries])
    if kind == "noalloc":
        out = state["out"]
        n = [G.gsmat_join_noalloc(store, pl, o.data_ptr(), o.shape[1], o.shape[1])
             for pl, o in zip(state["plans"], out)]
        return [np.array(n, np.int64), out]
    if kind == "fetch":
        pl = G.gsmat_plan(store, queries[0], mode)
        res = G.gsmat_join(store, pl)
        out = [G.gsmat_result_info(res)["rows"],
               G.gsmat_fetch_bindings(res, state["offset"], state["limit"])]
        res.close()
        pl.close()
        return out
    if kind == "count":
        infos, pages = np.zeros((len(queries), 2, 8), np.int64), []
        for i, q in enumerate(queries):
            pl = G.gsmat_plan(store, q, mode)
            res = G.gsmat_join(store, pl)
            info = G.gsmat_result_info(res)
            pages.append(G.gsmat_fetch_bindings(res, info["rows"] // 2, 1000))
            infos[i, 0, :len(info["step_rows_in"])] = info["step_rows_in"]
            infos[i, 1, :len(info["step_rows_out"])] = info["step_rows_out"]
            infos[i, :, 7] = info["rows"]
            res.close()
            pl.close()
        return [infos] + _gather(state["buf"], pages)
    if kind == "ext":
        out = []
        for pats, filters, nv in queries:
            res = G.gsmat_join_ext(store, pats, filters, nv)
            out.append(G.gsmat_fetch_bindings(res))
            res.close()
        return _gather(state["buf"], out)
    if kind == "batch":
        return _gather(state["buf"], G.evaluate_batch(store, queries, mode))
    if kind == "sweep":
        res, _ = G.gsmat_join_batch_bgp(store, state["packed"], mode, as_set=True)
        out = [res.rows()] + _gather(state["buf"],
                                     [G.gsmat_fetch_bindings(res[i]) for i in state["read"]])
        res.close()
        return out
    if kind == "serve":
        server, n = state["server"], len(queries)
        plans, _ = G.gsmat_plan_batch(store, queries, mode)
        for i, pl in enumerate(plans):
            G.gsmat_server_submit(server, pl, i)
        out, left = [None] * n, n
        while left:
            G.gsmat_server_step(server)
            for tag, res, _ in G.gsmat_server_poll(server, n):
                out[tag] = G.gsmat_fetch_bindings(res)
                res.close()
                left -= 1
        for pl in plans:
            pl.close()
        return _gather(state["buf"], out)
    raise ValueError(kind)


def _mean_rows(case):
    """Mean result size when sizes are spread evenly over the decades."""
    lo, hi = case["rows_lo"], max(case["rows_hi"], case["rows_lo"] + 1)
    return (hi - lo) / math.log(hi / lo)


def work(case):
    """Bytes of one pass: every binding written once (4 bytes per variable)
    and the member id that each row of the last step appends read once; a
    filter reads and a path's rows are written once; a build reads 12 bytes
    per triple and writes the two matrices (member lists, row ids, offsets)."""
    kind = case["kind"]
    if kind == "load_build":
        return {"bytes": case["triples"] * (12.0 + 4 * 3 + 2 * 4), "flops": 0.0}
    n = case["queries"]
    if kind == "cyclic":
        paths = math.sqrt(case["paths_lo"] * case["paths_hi"])
        return {"bytes": n * paths * 4.0 * case["nodes"], "flops": 0.0}
    if kind == "star":
        # the ids of the constants' lists: a hub of rank k is the object of the
        # share (1 / 3) V^(-1/3) k^(-2/3) of the triples that are not near ones,
        # a tenth of them along one of the frequent predicates
        g = GRAPHS[case["graph"]]
        k = sum(x ** (-2 / 3) for x in range(1, case["hub_rank"] + 1)) / case["hub_rank"]
        ids = 0.7 * g["T"] * 0.1 * k / 3 * g["V"] ** (-1 / 3)
        return {"bytes": n * case["members"] * 4.0 * ids, "flops": 0.0}
    cols = (case["pats_lo"] + case["pats_hi"]) / 2 + 0.5
    return {"bytes": n * _mean_rows(case) * 4.0 * (cols + 1), "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number and is compared as such; the order of
    an answer's rows is the library's own, so there is nothing to give."""
    return None
