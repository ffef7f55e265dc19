"""Workloads of the counting library, each one pass through its public entry points.

A case is a dict of plain values: the data graph (family, vertices, edges),
what is asked of it (``kind``), the pattern or patterns, where the plan comes from
(``config``: the cost model's choice, or a configuration that measured selection
keeps), how it counts (``iep``) and the launch fields a caller passes (0: the
plan's own). Graphs are drawn on the GPU from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2009_10955_amd import gp
from paper_2009_10955_amd import inputs as I

# Configurations that measured selection keeps on power-law graphs: schedule and
# restriction pairs (a, b), id(a) > id(b).
MEASURED = {
    "house": ((0, 1, 2, 3, 4), ((1, 0),)),
    "5-cycle": ((0, 1, 2, 3, 4), ((1, 0), (1, 2), (1, 3), (1, 4), (2, 0))),
    "4-clique": ((0, 1, 2, 3), ((0, 2), (0, 3), (1, 0), (1, 2), (1, 3), (3, 2))),
    "5-clique": ((0, 1, 2, 3, 4), ((0, 1), (0, 2), (0, 3), (0, 4), (1, 2), (1, 3), (1, 4), (2, 3), (2, 4), (3, 4))),
}

# Launch shapes that measured selection keeps for the patterns of a batch.
BATCH_SHAPES = {
    "6-cycle-chord": dict(group=16, chunk=1, split_vertices=1024),
    "prism": dict(group=16, chunk=1),
    "k4-path": dict(group=64, leaf_mode=3),
    "5-wheel": dict(group=32),
    "6-clique": dict(group=8),
}

LAUNCH = ("group", "leaf_mode", "chunk", "split_ways", "split_vertices", "root_stride", "root_offset")


def _case(name, kind, family, n, m, pattern="", **more):
    c = dict(kind=kind, family=family, n=n, m=m, pattern=pattern, config="model", iep=0, group=0, leaf_mode=0, chunk=0,
             split_ways=0, split_vertices=0, root_stride=0, root_offset=0, hubs="auto", capacity=0)
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # The smallest call: an exploratory count on a graph of a thousand
        # vertices, where launches, allocations and the wait are all there is.
        _case("er1000-4cycle", "count", "er", 1000, 5017, "4-cycle"),
        # Clustering statistics of a MiCo-sized power-law graph: the triangle
        # count, with the plan and launch that the library picks by itself.
        _case("rmat17-triangle", "count", "rmat", 131072, 971517, "triangle"),
        # The repeated query of the R-MAT 17 benchmark, as a program that tuned
        # its plans once keeps it: house with inclusion-exclusion ...
        _case("rmat17-house-iep", "count", "rmat", 131072, 971517, "house", config="measured", iep=1, group=32, chunk=2,
              split_ways=4, split_vertices=64),
        # ... the 5-cycle with long hub lists walked by whole groups ...
        _case("rmat17-5cycle", "count", "rmat", 131072, 971517, "5-cycle", config="measured", group=64, leaf_mode=4,
              chunk=4, split_ways=4, split_vertices=256),
        # ... and the 5-clique in narrow groups, enqueued without a wait.
        _case("rmat17-5clique", "async", "rmat", 131072, 971517, "5-clique", config="measured", group=16, chunk=2,
              split_ways=4, split_vertices=1024),
        # An ordinary count with nothing tuned, on a graph whose size is no
        # power of two: every 4-clique of half a million vertices.
        _case("rmat19-4clique", "count", "rmat", 400003, 3200000, "4-clique"),
        # A motif profile of a Wiki-Vote-sized graph: four 6-vertex patterns
        # counted together by one captured batch, replayed per query.
        _case("chunglu7000-batch", "batch", "chunglu", 7000, 99199, "prism+k4-path+5-wheel+6-clique"),
        # Edge features: how many 4-cliques hang on each edge.
        _case("rmat18-4clique-per-root", "per_root", "rmat", 262144, 1950000, "4-clique"),
        # A page of matches for a downstream program: rows of a 4-clique listing.
        _case("rmat16-4clique-list", "list", "rmat", 65536, 480000, "4-clique", capacity=12000000),
        # A new graph arrives: validation, layout, hub bitmaps, triangle count,
        # and the layout handed back.
        _case("rmat20-load", "load", "rmat", 1048576, 8000000),
        # A burst of small queries at the serving loop: every connected pattern
        # of three to five vertices on one resident graph.
        _case("chunglu3000-serve", "serve", "chunglu", 3000, 30000, "3..5"),
        # The largest: one strided slice of the house count on a
        # LiveJournal-sized graph, as a long count is cut into steps.
        _case("rmat22-house-slice", "count", "rmat", 4194304, 32621008, "house", config="measured", iep=1, group=64, chunk=4,
              split_ways=16, split_vertices=256, root_stride=60, root_offset=7),
    ]


# Most edges on which a pattern is counted, by graph family: beyond these
# one count takes longer than the largest listed case.
MOST_M = {
    "rmat": {"triangle": 1 << 23, "4-clique": 1 << 22, "5-clique": 1 << 20, "diamond": 1 << 20, "4-cycle": 1 << 19,
             "tailed-triangle": 1 << 20, "house": 1 << 20, "5-cycle": 1 << 18, "4-star": 1 << 21, "4-path": 1 << 19},
    "chunglu": {"prism": 100000, "k4-path": 100000, "5-wheel": 100000, "6-clique": 100000, "house": 100000,
                "5-cycle": 60000, "4-cycle": 100000, "5-path": 100000, "6-cycle": 15000, "6-cycle-chord": 40000},
    "er": {"triangle": 60000, "4-cycle": 60000, "house": 60000, "5-cycle": 60000},
}
IEP_ONLY = ("4-star", "4-path", "5-path")  # trees: counted with inclusion-exclusion, as the serving loop does


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["count"] * 5 + ["async", "per_root", "list", "load", "batch", "serve"])
    if kind == "serve":
        n = _log_int(rng, 300, 3000)
        return _case(None, kind, "chunglu", n, int(n * rng.uniform(5, 10)), "3..%d" % rng.choice([4, 5]))
    if kind == "batch":
        n = _log_int(rng, 1000, 7000)
        pats = sorted(rng.sample(["prism", "k4-path", "5-wheel", "6-clique"], rng.choice([2, 3, 4])))
        return _case(None, kind, "chunglu", n, int(n * rng.uniform(6, 14)), "+".join(pats))
    if kind == "load":
        n = _log_int(rng, 1000, 1000000)
        family = "rmat" if n > 8000 else rng.choice(["rmat", "chunglu", "er"])
        return _case(None, kind, family, n, int(n * rng.uniform(4, 8)), hubs=rng.choice(["auto", "auto", "none"]))
    if kind == "list":
        n = _log_int(rng, 2000, 65000)
        return _case(None, kind, "rmat", n, int(n * rng.uniform(5, 8)), rng.choice(["triangle", "4-clique", "diamond"]),
                     capacity=_log_int(rng, 10000, 4000000))
    family = rng.choice(["rmat", "rmat", "chunglu", "er"])
    pattern = rng.choice(sorted(MOST_M[family]))
    most = MOST_M[family][pattern]
    m = _log_int(rng, min(2000, most // 4), most)
    n = max(100, int(m / (rng.uniform(8, 20) if family == "er" else rng.uniform(4, 14))))
    c = _case(None, kind, family, n, m, pattern, hubs=rng.choice(["auto"] * 5 + ["none"]) if m <= most // 8 else "auto")
    if pattern in IEP_ONLY or (pattern == "house" and rng.random() < 0.6):
        c["iep"] = 1
    if pattern in MEASURED and family == "rmat":
        c["config"] = "measured"
    if rng.random() < 0.6:  # a caller's own launch shape
        c["group"] = rng.choice([64, 32, 16])
        c["leaf_mode"] = rng.choice([1, 1, 3, 4])
        c["chunk"] = rng.choice([1, 2, 4, 8])
        c["split_ways"] = rng.choice([1, 4, 16])
    if kind != "per_root" and family != "er" and rng.random() < 0.2:
        c["root_stride"] = rng.choice([3, 7, 20])
        c["root_offset"] = rng.randrange(c["root_stride"])
    return c


# ------------------------------------------------------------------ graphs

def _rmat(n, count, gen):
    """Edges u < v as keys u * n + v: R-MAT (.57, .19, .19, .05) draws."""
    scale = max(1, (n - 1).bit_length())
    keys = []
    for done in range(0, count, 1 << 23):
        cnt = min(1 << 23, count - done)
        u = torch.zeros(cnt, dtype=torch.int64, device="cuda")
        v = torch.zeros_like(u)
        for _ in range(scale):
            r = torch.rand(cnt, generator=gen, device="cuda")
            u = 2 * u + (r >= 0.76)
            v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
        keep = (u != v) & (u < n) & (v < n)
        u, v = u[keep], v[keep]
        keys.append(torch.minimum(u, v) * n + torch.maximum(u, v))
    return torch.cat(keys)


def _weighted(n, count, gen, m, family):
    """The same with both endpoints drawn by weight: uniform, or Chung-Lu with
    exponent 2.1, weights capped at the root of their sum."""
    w = np.ones(n)
    if family == "chunglu":
        w = np.arange(1, n + 1, dtype=np.float64) ** (-1.0 / 1.1)
        for _ in range(100):
            w *= 2.0 * m / w.sum()
            if w.max() <= math.sqrt(2.0 * m) * (1 + 1e-12):
                break
            w = np.minimum(w, math.sqrt(2.0 * m))
    cum = torch.from_numpy(np.cumsum(w) / w.sum()).cuda()
    ends = torch.searchsorted(cum, torch.rand((2, count), generator=gen, device="cuda", dtype=torch.float64))
    u, v = ends.clamp_(max=n - 1)
    keep = u != v
    u, v = u[keep], v[keep]
    return torch.minimum(u, v) * n + torch.maximum(u, v)


def _csr(case, seed):
    """(row_ptr int64, col int32) on the GPU: exactly m distinct edges, sorted
    lists, both directions."""
    n, m = case["n"], case["m"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    key = torch.zeros(0, dtype=torch.int64, device="cuda")
    while key.numel() < m:
        more = int(1.15 * (m - key.numel())) + 1000
        if case["family"] == "rmat":
            drawn = _rmat(n, more, gen)
        else:
            drawn = _weighted(n, more, gen, m, case["family"])
        key = torch.unique(torch.cat([key, drawn]))
    key = key[torch.randperm(key.numel(), generator=gen, device="cuda")[:m]]
    a, b = key // n, key % n
    both = torch.sort(torch.cat([key, b * n + a])).values
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(both // n, minlength=n), 0, out=row_ptr[1:])
    return row_ptr, (both % n).to(torch.int32)


# ------------------------------------------------------------------- a pass

def _plan(case, pattern, stats):
    k, edges = I.PATTERNS[pattern]
    opts = {}
    if case["config"] == "measured":
        opts = dict(force_order=MEASURED[pattern][0], force_restr=MEASURED[pattern][1])
    return gp.Plan(k, edges, stats=stats, iep=bool(case["iep"]), **opts)


def prepare(case, seed):
    row_ptr, col = _csr(case, seed)
    s = {"case": case, "kind": case["kind"], "launch": {f: case[f] for f in LAUNCH if case[f]}}
    if s["kind"] == "load":
        s["csr"] = (row_ptr, col)
        return s
    graph = s["graph"] = gp.Graph(row_ptr, col, hub_bitmaps=case["hubs"])
    if s["kind"] == "serve":
        most = int(case["pattern"].split("..")[1])
        s["queries"] = list(I.connected_patterns(3, most))
        np.random.default_rng(seed).shuffle(s["queries"])
        s["server"] = gp.Server([graph])
    elif s["kind"] == "batch":
        names = case["pattern"].split("+")
        s["plans"] = [_plan(case, p, graph.stats()).with_launch(**BATCH_SHAPES[p]) for p in names]
        s["batch"] = gp.Batch(graph, s["plans"], batch_runs=2)
    else:
        s["plan"] = _plan(case, case["pattern"], graph.stats())
        if s["kind"] == "async":
            s["out"] = torch.zeros(2, dtype=torch.int64, device="cuda")
        elif s["kind"] == "list":
            s["out"] = torch.zeros((case["capacity"], s["plan"].k), dtype=torch.int32, device="cuda")
    return s


def run(s):
    kind = s["kind"]
    if kind == "count":
        return gp.count(s["graph"], s["plan"], **s["launch"])
    if kind == "async":
        gp.count_async(s["graph"], s["plan"], s["out"], **s["launch"])
        return s["out"]
    if kind == "per_root":
        return gp.count_per_root(s["graph"], s["plan"], **s["launch"])
    if kind == "list":
        _, total = gp.list_embeddings(s["graph"], s["plan"], capacity=s["case"]["capacity"], out=s["out"], **s["launch"])
        return s["out"], total
    if kind == "batch":
        return s["batch"].run()
    if kind == "serve":
        tickets = [s["server"].submit(0, k, edges) for k, edges in s["queries"]]
        return [s["server"].wait(t)[:2] for t in tickets]
    graph = gp.Graph(*s["csr"], hub_bitmaps=s["case"]["hubs"])
    st = graph.stats()
    row_ptr, col = graph.layout()
    out = {"tri_cnt": st.tri_cnt, "max_degree": st.max_degree, "hub_vertices": st.hub_vertices, "new_id": graph.new_id(),
           "row_ptr": row_ptr, "col": col}
    graph.close()
    return out


def work(case):
    """The graph read once as sorted lists and root edges, the result written
    once. What a count intersects beyond that depends on the graph drawn."""
    n, m, kind = case["n"], case["m"], case["kind"]
    graph = 8 * (n + 1) + 4 * 2 * m
    roots = 8 * m / max(1, case["root_stride"])
    out = 8
    if kind == "load":
        return {"bytes": 2 * graph + 4 * n, "flops": 0}
    if kind == "per_root":
        out = 8 * 2 * m
    elif kind == "list":
        out = 4 * I.PATTERNS[case["pattern"]][0] * case["capacity"]
    return {"bytes": graph + roots + out, "flops": 0}


# -------------------------------------------------------------------- exact

def _dense_count(pattern, a):
    """Closed forms over the adjacency matrix a (float64, exact integers)."""
    common = a @ a
    if pattern == "triangle":
        return int((common * a).sum().item()) // 6
    pairs = common * (common - 1) / 2
    if pattern == "diamond":
        return int((pairs * a).sum().item()) // 2
    pairs.fill_diagonal_(0)
    return int(pairs.sum().item()) // 4  # 4-cycle: each found from both of its diagonals, in both orders


def exact(case, seed):
    if case["kind"] == "load" and case["m"] <= 2000000:
        row_ptr, col = (t.cpu().numpy() for t in _csr(case, seed))
        deg = np.diff(row_ptr)
        order = np.argsort(-deg, kind="stable")
        new_id = np.empty(case["n"], dtype=np.int32)
        new_id[order] = np.arange(case["n"], dtype=np.int32)
        keys = np.sort(np.repeat(new_id, deg).astype(np.int64) * case["n"] + new_id[col])
        return {"tri_cnt": None, "max_degree": int(deg.max()), "hub_vertices": None, "new_id": new_id,
                "row_ptr": np.concatenate([[0], np.cumsum(deg[order])]), "col": (keys % case["n"]).astype(np.int32)}
    if case["kind"] in ("count", "async") and case["n"] <= 4000 and not case["root_stride"] \
            and case["pattern"] in ("triangle", "diamond", "4-cycle"):
        row_ptr, col = _csr(case, seed)
        a = torch.zeros((case["n"], case["n"]), dtype=torch.float64)
        rows = torch.repeat_interleave(torch.arange(case["n"]), torch.diff(row_ptr).cpu())
        a[rows, col.cpu().long()] = 1.0
        c = _dense_count(case["pattern"], a)
        return c if case["kind"] == "count" else torch.tensor([c, 0], dtype=torch.int64)
    return None
