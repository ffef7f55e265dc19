"""Rules that pick a kernel or a launch from the plan and the graph: which side of
them a graph falls on, and the same counts on both. Counts are integers: every
comparison is exact."""
import itertools
import random

import numpy as np
import pytest

import oracle as O
from paper_2009_10955_amd import gp
from paper_2009_10955_amd import inputs as I

pytestmark = pytest.mark.gpu
P = I.PATTERNS
# the path-table form of these patterns, and the house with inclusion-exclusion
HOUSE = dict(force_order=(0, 1, 2, 3, 4), force_restr=[(1, 0)], iep=True)
FIVE = dict(force_order=(0, 1, 2, 3, 4), force_restr=[(1, 0), (1, 2), (1, 3), (1, 4), (2, 0)])


def _uniform(n, m, seed=1):
    rng = np.random.default_rng(seed)
    return I.csr_from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m))


def _torus(w):
    x = np.arange(w * w)
    r, c = x // w, x % w
    return I.csr_from_edges(w * w, np.concatenate([x, x]), np.concatenate([r * w + (c + 1) % w, (r + 1) % w * w + c]))


def _hubs(n, m, hubs, deg, seed=1):
    """A uniform graph with hubs of degree deg."""
    rng = np.random.default_rng(seed)
    src = np.concatenate([rng.integers(0, n, m), np.repeat(np.arange(hubs), deg)])
    dst = np.concatenate([rng.integers(0, n, m), rng.integers(0, n, hubs * deg)])
    return I.csr_from_edges(n, src, dst)


def _orders(k, edges):
    adj = {(a, b) for a, b in edges} | {(b, a) for a, b in edges}
    return [o for o in itertools.permutations(range(k))
            if all(any((o[i], o[j]) in adj for j in range(i)) for i in range(1, k))]


# ------------------------------------------------------- path table or general search

@pytest.mark.parametrize("g", [_uniform(20000, 160000), _uniform(100000, 400000), _torus(300)],
                         ids=["G20000", "G100000", "torus"])
@pytest.mark.parametrize("pname,opts", [("4-cycle", {}), ("5-cycle", {}), ("5-cycle", FIVE), ("house", HOUSE)])
def test_no_path_table_where_degrees_are_small_and_even(g, pname, opts):
    """A fill of the table per root edge costs more than the search there (5-cycle on
    the torus of 1M vertices 26 ms with tables, 1.2 without)."""
    graph = gp.Graph.from_csr(g, device=True)
    plan = gp.Plan(*P[pname], stats=graph.stats(), **opts)
    assert gp.count_shape(graph, plan)["table"] == 0
    assert gp.count(graph, plan) == gp.count_per_root(graph, plan)[0]
    graph.close()


@pytest.mark.parametrize("pname,n,m,hubs,deg", [("4-cycle", 3000, 9000, 30, 900), ("4-cycle", 8193, 30000, 30, 1500),
                                                ("5-cycle", 8192, 20000, 8, 900), ("5-cycle", 8193, 20000, 8, 1500),
                                                ("5-cycle", 40000, 60000, 6, 3000), ("6-cycle", 9000, 9000, 3, 500)])
def test_path_table_kernels_count_as_the_general_search(pname, n, m, hubs, deg):
    """Graphs on the table's side of the rule, with fewer vertices than the table holds,
    one more and many more: counted whole, sampled, in a batch, with accounting,
    against the general search (per-root counts never use the table), over schedules
    and sets that leave an endpoint out of the table or fill it anew at every root."""
    k, e = P[pname]
    rnd = random.Random(n)
    orders = _orders(k, e)
    for bits in ("auto", "none"):
        graph = gp.Graph.from_csr(_hubs(n, m, hubs, deg), device=True, hub_bitmaps=bits)
        st = graph.stats()
        plans = [gp.Plan(k, e, stats=st)]
        for _ in range(400):
            if len(plans) == 6:
                break
            p = gp.Plan(k, e, stats=st, force_order=rnd.choice(orders), force_set=rnd.randrange(plans[0].info().n_sets))
            if gp.count_shape(graph, p)["table"]:
                plans.append(p)
        assert len(plans) == 6 and gp.count_shape(graph, plans[0])["table"]
        want = gp.count_per_root(graph, plans[0])[0]
        for p in plans:
            assert gp.count(graph, p) == want, (bits, p.order, p.restrictions)
            assert sum(gp.count(graph, p, root_stride=5, root_offset=o) for o in range(5)) == want
            assert gp.count_traffic(graph, p)[0] == want
        assert gp.count_batch(graph, plans, batch_runs=2) == [want] * 6
        graph.close()


@pytest.mark.parametrize("n", [3000, 16385, 40000])
def test_iep_table_kernel_counts_as_the_general_search(n):
    """The house by the inclusion-exclusion table, with vertices below and past its end."""
    graph = gp.Graph.from_csr(_hubs(n, 2 * n, 12, n // 4), device=True)
    plan = gp.Plan(*P["house"], stats=graph.stats(), **HOUSE)
    shape = gp.count_shape(graph, plan)
    assert shape["table"] == 1 and shape["threads"] == 512 and plan.info().iep == 2
    want = gp.count_per_root(graph, plan)[0]
    assert gp.count(graph, plan) == want
    assert gp.count_traffic(graph, plan)[0] == want
    graph.close()


def test_tables_against_the_oracle():
    """The 5-cycle against the oracle, the 4-cycle against its closed form over the
    adjacency matrix, both counted with tables."""
    g = _hubs(600, 1500, 6, 250)
    graph = gp.Graph.from_csr(g, device=True)
    for opts in ({}, FIVE):
        plan = gp.Plan(*P["5-cycle"], stats=graph.stats(), **opts)
        assert gp.count_shape(graph, plan)["table"] == 1
        assert gp.count(graph, plan) == O.count(g, *P["5-cycle"])
    graph.close()
    g = _hubs(2000, 6000, 40, 700)
    a = np.zeros((2000, 2000))
    a[np.repeat(np.arange(2000), g.degrees()), g.col] = 1
    common = a @ a
    np.fill_diagonal(common, 0)
    graph = gp.Graph.from_csr(g, device=True)
    plan = gp.Plan(*P["4-cycle"], stats=graph.stats())
    assert gp.count_shape(graph, plan)["table"] == 1
    assert gp.count(graph, plan) == int((common * (common - 1) / 2).sum()) // 4
    graph.close()


# ------------------------------------------------------- width and grab of a default launch

def _power_law(n=20000, m=60000, seed=3):
    """Endpoints drawn by weight i^-0.9: a few hundred hubs over short lists."""
    rng = np.random.default_rng(seed)
    w = np.minimum(np.arange(1, n + 1) ** -0.9, 0.01 * (np.arange(1, n + 1) ** -0.9).sum())
    cum = np.cumsum(w) / w.sum()
    return I.csr_from_edges(n, *np.minimum(np.searchsorted(cum, rng.random((2, m))), n - 1))


@pytest.mark.parametrize("pname,order,fs,want", [
    ("5-cycle", (0, 1, 2, 4, 3), 8, (16, 1)),   # level-2 candidates a whole list: single tasks
    ("house", (1, 4, 2, 3, 0), 2, (16, 1)),
    ("house", (4, 1, 0, 2, 3), 0, (32, 2)),     # a built set, then the hub's whole list over the lanes
    ("5-clique", None, 0, (16, 4)),             # built sets all the way
    ("4-clique", None, 0, (16, 4)),
])
def test_heavy_roots_set_width_and_grab(pname, order, fs, want):
    """Groups of 16 lanes that take four heavy roots at once end last: 5-cycle of schedule
    0,1,2,4,3 on R-MAT (131,072 vertices, 200K edges) 301 ms, 100 one at a time."""
    k, e = P[pname]
    for g, expect in ((_power_law(), want), (_uniform(20000, 60000), (16, 4))):
        graph = gp.Graph.from_csr(g, device=True)
        opts = dict(force_order=order, force_set=fs) if order else {}
        plan = gp.Plan(k, e, stats=graph.stats(), **opts)
        s = gp.count_shape(graph, plan)
        assert (s["table"], s["group"], s["chunk"]) == (0,) + expect, pname
        # a caller's own choice stays
        s = gp.count_shape(graph, plan, group=16)
        assert (s["group"], s["chunk"]) == (16, 4)
        assert gp.count_shape(graph, plan, chunk=8)["chunk"] == 8
        n = gp.count(graph, plan)
        assert n == gp.count(graph, plan, group=64) == gp.count_per_root(graph, plan)[0]
        assert gp.count_batch(graph, [plan, plan]) == [n, n]
        graph.close()


# ------------------------------------------------------- loading

def test_bitmaps_do_not_evict_the_runtimes_freed_blocks():
    """Loading and freeing a graph with 47 MB of bitmaps beside 38 MB of arrays, against
    the same graph without bitmaps: they cost 0.3 ms, and 1.9 where the runtime gave all
    of the graph's blocks back (the fastest of 15 passes each)."""
    import time
    import torch
    g = _power_law(150000, 900000)
    rp, col = torch.from_numpy(g.row_ptr).cuda(), torch.from_numpy(g.col).cuda()
    best = {}
    for bits in ("auto", "none"):
        for _ in range(16):
            torch.cuda.synchronize()
            t = time.perf_counter()
            graph = gp.Graph(rp, col, hub_bitmaps=bits)
            size = graph.stats().hub_bitmap_bytes
            graph.close()
            best[bits] = min(best.get(bits, 1.0), time.perf_counter() - t)
        assert (size > 32 << 20) == (bits == "auto")
    assert best["auto"] - best["none"] < 1e-3, best


# ------------------------------------------------------- estimates and tuning of table plans

@pytest.fixture(scope="module")
def rmat16():
    graph = gp.Graph.from_csr(I.rmat(16, 8, seed=5), device=True)
    yield graph
    graph.close()


@pytest.mark.parametrize("pname,opts", [("4-cycle", {}), ("5-cycle", {}), ("5-cycle", FIVE), ("house", HOUSE)])
def test_estimates_measure_the_kernel_that_counts(rmat16, pname, opts):
    """Sampled roots fill a table each, where a whole count fills one for a run of roots,
    and with inclusion-exclusion sparse samples ran on the other kernel: estimates of
    these counts, 2 to 60 ms, were 5 to 15 times too high. They are within 4 either way."""
    import time
    plan = gp.Plan(*P[pname], stats=rmat16.stats(), **opts)
    assert gp.count_shape(rmat16, plan)["table"] == 1
    ms = 1e9
    for _ in range(3):
        gp.count(rmat16, plan)
        t = time.perf_counter()
        gp.count(rmat16, plan)
        ms = min(ms, 1e3 * (time.perf_counter() - t))
        est = gp.estimate(rmat16, plan)
    assert ms / 4 <= est["ms"] <= 4 * ms, (pname, ms, est)


def test_tuning_keeps_the_default_shape_of_table_plans():
    """Every shape of such a plan is one launch: the tuner measured them all and kept what
    noise picked, for the per-root counts and batches that do not use the table too."""
    graph = gp.Graph.from_csr(_hubs(8000, 20000, 20, 1500), device=True)
    plan = gp.Plan(*P["5-cycle"], stats=graph.stats())
    tuned = plan.tuned(graph, max_configs=6, budget_seconds=0.5)
    assert gp.count_shape(graph, tuned)["table"] == 1
    skip = ("waves_per_cu",)
    assert {k: v for k, v in tuned.launch().items() if k not in skip} == \
           {k: v for k, v in plan.launch().items() if k not in skip}
    assert gp.count(graph, tuned) == gp.count(graph, plan)
    graph.close()


# ------------------------------------------------------- batches

def test_batches_follow_the_sampling_rule():
    """A batch set to a sparse sample with inclusion-exclusion leaves the table, as a count
    of that sample does, and takes it again; counts are those of the samples."""
    graph = gp.Graph.from_csr(_hubs(3000, 6000, 12, 2500), device=True)
    st = graph.stats()
    plans = [gp.Plan(*P["house"], stats=st, **HOUSE), gp.Plan(*P["4-clique"], stats=st),
             gp.Plan(*P["5-cycle"], stats=st)]
    batch = gp.Batch(graph, plans)
    sparse = st.max_degree // 1024 + 1
    for stride, offset in ((1, 0), (sparse, 1), (64, 5), (1, 0), (sparse, 0), (1, 0)):
        batch.set_sample(stride, offset)
        la = dict(root_stride=stride, root_offset=offset)
        for i, p in enumerate(plans):
            assert batch.shape(i)["table"] == gp.count_shape(graph, p, **la)["table"], (stride, i)
        assert batch.shape(0)["table"] == (stride == 1) and batch.shape(1)["table"] == 0
        for _ in range(2):
            assert batch.run() == [gp.count(graph, p, **la) for p in plans], stride
    batch.close()
    graph.close()


# ------------------------------------------------------- serving

def test_admission_estimates_what_is_served(rmat16):
    """With max_query_ms a query's slices run on the general search, also where a whole
    count of its plan runs on path tables, ten times faster: a limit between the two
    refuses it, and one above both serves it."""
    plan = gp.Plan(*P["5-cycle"], stats=rmat16.stats())
    assert gp.count_shape(rmat16, plan)["table"] == 1
    table_ms = gp.estimate(rmat16, plan)["ms"]
    for limit, want in ((3 * table_ms, -10), (100 * table_ms, 0)):
        srv = gp.Server([rmat16], max_query_ms=limit)
        status, count, _ = srv.wait(srv.submit(0, *P["5-cycle"]))
        srv.close()
        assert status == want, (limit, status)
        if want == 0:
            assert count == gp.count(rmat16, plan)


# ------------------------------------------------------- the general search's paths, off the tables

# 5-vertex patterns whose last level is N(x) & N(root endpoint), cut by root levels, below
# a set that is built at the root: leaf mode 4 keeps its sizes, path tables do not take it
MEMO_PLANS = [
    ([(0, 1), (0, 2), (0, 3), (0, 4), (1, 2), (1, 4), (2, 3)], (4, 0, 1, 2, 3), 2),
    ([(0, 2), (0, 3), (0, 4), (1, 2), (1, 3), (1, 4), (2, 3)], (0, 2, 3, 1, 4), 0),
    ([(0, 2), (0, 3), (0, 4), (1, 2), (1, 3), (1, 4), (2, 3)], (2, 1, 3, 0, 4), 0),
    ([(0, 1), (0, 2), (0, 3), (0, 4), (1, 2), (1, 3), (1, 4), (2, 3)], (2, 0, 3, 1, 4), 0),
]


@pytest.mark.parametrize("edges,order,fs", MEMO_PLANS, ids=range(len(MEMO_PLANS)))
def test_leaf4_memo_on_plans_without_a_table(edges, order, fs):
    """Leaf mode 4's sizes per root, with hits (a candidate comes up below several level-2
    bindings of a root): every grab, split and width, with every vertex a hub and with hubs
    by degree, counted, accounted, without allocation and in a batch: the oracle's
    count."""
    import torch
    g = I.er(120, 0.3, seed=5)
    want = O.count(g, 5, edges)
    for bits in ("dense", "auto"):
        graph = gp.Graph.from_csr(g, device=True, hub_bitmaps=bits)
        plan = gp.Plan(5, edges, stats=graph.stats(), force_order=order, force_set=fs)
        for ch in (1, 4, 16):
            for sw, sv in ((1, 0), (16, 1 << 20), (3, 8)):
                for grp in (64, 32, 16, 8):
                    la = dict(group=grp, leaf_mode=4, chunk=ch, split_ways=sw, split_vertices=sv)
                    s = gp.count_shape(graph, plan, **la)
                    assert (s["table"], s["group"]) == (0, grp)
                    assert s["memo"] == (graph.stats().hub_vertices > 0)
                    assert gp.count(graph, plan, **la) == want, (bits, la)
        assert gp.count_traffic(graph, plan, group=64, leaf_mode=4)[0] == want
        out = torch.zeros(2, dtype=torch.int64, device="cuda")
        gp.count_noalloc(graph, plan, out, group=64, leaf_mode=4)
        torch.cuda.synchronize()
        assert out.tolist() == [want, 0]
        assert gp.count_batch(graph, [plan, plan, plan], group=32, leaf_mode=4) == [want] * 3
        graph.close()


@pytest.mark.parametrize("pname", ["4-cycle", "5-cycle", "6-cycle"])
def test_cycles_off_the_tables(pname):
    """Schedules and sets of the cycles that path tables do not take, over every width, leaf
    mode and split, per root too: the oracle's count, by the general search."""
    k, e = P[pname]
    g = I.er(48, 0.3, seed=21)
    want = O.count(g, k, e)
    rnd = random.Random(k)
    orders, n_sets = _orders(k, e), gp.Plan(k, e).info().n_sets
    for bits in ("dense", "none"):
        graph = gp.Graph.from_csr(g, device=True, hub_bitmaps=bits)
        plans = []
        for _ in range(400):
            p = gp.Plan(k, e, stats=graph.stats(), force_order=rnd.choice(orders), force_set=rnd.randrange(n_sets))
            if not gp.count_shape(graph, p)["table"]:
                plans.append(p)
            if len(plans) == 4:
                break
        assert len(plans) == 4
        for p in plans:
            for grp, leaf in itertools.product((64, 32, 16, 8), (1, 2, 3, 4)):
                la = dict(group=grp, leaf_mode=leaf, chunk=rnd.choice((1, 3, 4)), split_ways=rnd.choice((1, 5, 16)),
                          split_vertices=rnd.choice((8, 1 << 20)))
                assert gp.count(graph, p, **la) == want, (bits, p.order, p.restrictions, la)
            assert gp.count_per_root(graph, p, group=16, leaf_mode=4)[0] == want
        graph.close()
