"""Paths of the counting kernels that depend on sizes and plan forms: the
inclusion-exclusion leaf over many schedules and restriction sets, the path
table and what lies past its end, root runs of one hub, the task queue's ends,
result slots shared by threads. Counts are integers: every comparison is exact."""
import itertools
import random
import threading

import numpy as np
import pytest

import oracle as O
from paper_2009_10955_amd import gp
from paper_2009_10955_amd import inputs as I

pytestmark = pytest.mark.gpu
P = I.PATTERNS


def _hub_graph(n=300, hubs=4, deg=150, rest=300, seed=7):
    """A few hubs with shared neighbourhoods (lists longer than a lane walks
    alone) over a sparse rest, so that wavefronts mix long walks and idle lanes."""
    rng = np.random.default_rng(seed)
    src, dst = [], []
    for h in range(hubs):
        nb = rng.choice(np.arange(hubs, n), size=deg, replace=False)
        src += [h] * deg + [h] * (hubs - 1 - h)
        dst += list(nb) + list(range(h + 1, hubs))
    src += list(rng.integers(hubs, n, rest))
    dst += list(rng.integers(hubs, n, rest))
    return I.csr_from_edges(n, np.array(src), np.array(dst))


def _orders(k, edges):
    """Every vertex order whose prefixes are connected."""
    adj = {(a, b) for a, b in edges} | {(b, a) for a, b in edges}
    return [o for o in itertools.permutations(range(k))
            if all(any((o[i], o[j]) in adj for j in range(i)) for i in range(1, k))]


def _configs(k, edges, many, seed):
    """Random (schedule, restriction set) pairs of a pattern."""
    rnd = random.Random(seed)
    n_sets = gp.Plan(k, edges).info().n_sets
    orders = _orders(k, edges)
    return [(rnd.choice(orders), rnd.randrange(n_sets)) for _ in range(many)]


@pytest.mark.parametrize("pname", ["house", "spider", "k4-path", "6-cycle-chord", "5-path", "4-path", "diamond"])
def test_iep_every_depth_over_schedules_and_sets(pname):
    """Subset sizes with one to four operands, equal subsets, sums taken apart,
    the table and the memo: whatever the schedule, set, depth, width and split,
    the count is the oracle's."""
    k, e = P[pname]
    g = _hub_graph()
    want = O.count(g, k, e)
    rnd = random.Random(3)
    for hubs in ("auto", "none", "dense"):
        graph = gp.Graph.from_csr(g, device=True, hub_bitmaps=hubs)
        seen = 0
        for order, fs in _configs(k, e, 16, seed=11):
            for n in (2, 3, 4):
                plan = gp.Plan(k, e, stats=graph.stats(), force_order=order, force_set=fs, iep=n)
                if plan.info().iep != n:
                    continue
                seen += 1
                la = dict(group=rnd.choice([64, 32]), chunk=rnd.choice([0, 1, 5]), split_ways=rnd.choice([1, 3, 16]),
                          split_vertices=rnd.choice([8, 1 << 20]))
                assert gp.count(graph, plan, **la) == want, (hubs, order, fs, n, la)
                if plan.info().iep_div == 1:
                    parts = [gp.count(graph, plan, root_stride=3, root_offset=o) for o in range(3)]
                    assert sum(parts) == want, (hubs, order, fs, n)
        assert seen > 0
        graph.close()


@pytest.mark.parametrize("pname,n,m", [("4-cycle", 700, 2500), ("4-cycle", 8193, 30000), ("5-cycle", 8192, 20000),
                                       ("5-cycle", 8193, 20000), ("5-cycle", 40000, 80000), ("6-cycle", 9000, 14000)])
def test_path_table_to_its_end_and_past_it(pname, n, m):
    """Plans whose last level is N(x) & N(root endpoint), with fewer vertices
    than the table holds, one more, and many more: the oracle's count, per root,
    sampled and in a batch, for schedules and sets that leave a root endpoint
    out of the table or fill it anew at every root."""
    k, e = P[pname]
    rng = np.random.default_rng(n)
    hub = rng.integers(0, n, (3, 120))  # three hubs beside the random edges
    src = np.concatenate([rng.integers(0, n, m), np.repeat(np.arange(3), 120)])
    dst = np.concatenate([rng.integers(0, n, m), hub.ravel()])
    g = I.csr_from_edges(n, src, dst)
    want = O.count(g, k, e)
    for hubs in ("auto", "none"):
        graph = gp.Graph.from_csr(g, device=True, hub_bitmaps=hubs)
        plans = [gp.Plan(k, e, stats=graph.stats())]
        plans += [gp.Plan(k, e, stats=graph.stats(), force_order=o, force_set=s) for o, s in _configs(k, e, 6, seed=n)]
        for p in plans:
            assert gp.count(graph, p) == want, (hubs, p.order, p.restrictions)
            assert gp.count_per_root(graph, p)[0] == want
            assert sum(gp.count(graph, p, root_stride=5, root_offset=o) for o in range(5)) == want
            assert gp.count_traffic(graph, p)[0] == want
        assert gp.count_batch(graph, plans[:3], batch_runs=2) == [want] * 3
        graph.close()


@pytest.mark.parametrize("n", [16385, 20000])
def test_iep_table_past_its_end(n):
    """The house with vertices past the table of the inclusion-exclusion kernel
    (their lists are walked against the filter of the hub's list)."""
    k, e = P["house"]
    rng = np.random.default_rng(n)
    hub = rng.integers(0, n, (4, 400))
    src = np.concatenate([rng.integers(0, n, 30000), np.repeat(np.arange(4), 400)])
    dst = np.concatenate([rng.integers(0, n, 30000), hub.ravel()])
    g = I.csr_from_edges(n, src, dst)
    want = O.count(g, k, e)
    for hubs in ("auto", "none"):
        graph = gp.Graph.from_csr(g, device=True, hub_bitmaps=hubs)
        plan = gp.Plan(k, e, stats=graph.stats(), force_order=(0, 1, 2, 3, 4), force_restr=[(1, 0)], iep=True)
        assert plan.info().iep == 2
        assert gp.count(graph, plan) == want
        assert gp.count_traffic(graph, plan)[0] == want
        assert sum(gp.count(graph, plan, root_stride=7, root_offset=o) for o in range(7)) == want
        assert gp.count_batch(graph, [plan, plan], batch_runs=2) == [want] * 2
        graph.close()


@pytest.mark.parametrize("m", [1, 15, 16, 17, 63, 64, 65, 1023, 1025])
def test_queue_hands_out_every_task_once(m):
    """Numbers of root tasks around the queue's cursors, a group's width and a
    grab, over grabs and widths: a path of m edges has m edges, m - 1 wedges."""
    v = np.arange(m)
    graph = gp.Graph.from_csr(I.csr_from_edges(m + 1, v, v + 1), device=True)
    for pname, want in (("edge", m), ("4-path", max(0, m - 2))):
        for iep in (False, True):
            plan = gp.Plan(*P[pname], stats=graph.stats(), iep=iep)
            for la in (dict(), dict(chunk=1), dict(chunk=7, group=16), dict(group=8, chunk=3), dict(xcd_tasks=4)):
                assert gp.count(graph, plan, **la) == want, (pname, iep, la)
    assert gp.list_embeddings(graph, gp.Plan(*P["4-path"], stats=graph.stats()))[1] == max(0, m - 2)
    graph.close()


@pytest.mark.parametrize("hubs", ["auto", "dense", "none"])
def test_isolated_vertices_have_no_bitmap_columns(hubs):
    """Most vertices isolated, at both ends of the id range: bitmaps end at the
    last vertex with a neighbor."""
    core = I.er(90, 0.5, seed=2)
    src = np.repeat(np.arange(core.n), core.degrees()) + 1000
    g = I.csr_from_edges(3000, src, core.col.astype(np.int64) + 1000)
    graph = gp.Graph.from_csr(g, device=True, hub_bitmaps=hubs)
    for pname in ("triangle", "4-clique", "4-cycle", "house", "5-clique"):
        for iep in (False, True):
            plan = gp.Plan(*P[pname], stats=graph.stats(), iep=iep)
            assert gp.count(graph, plan) == O.count(core, *P[pname]), (pname, iep)
    graph.close()


def test_threads_share_a_graph():
    """Blocking counts from several threads, each on its own stream: the
    graph's result slots and the pool serve them all, and a graph counted after
    every other was freed starts over."""
    import torch
    g = I.er(400, 0.05, seed=4)
    names = ["triangle", "4-cycle", "house", "5-cycle"]
    want = {x: O.count(g, *P[x]) for x in names}
    for _ in range(2):
        graph = gp.Graph.from_csr(g, device=True)
        plans = {x: gp.Plan(*P[x], stats=graph.stats(), iep=x == "house") for x in names}
        bad = []

        def work(i):
            torch.cuda.set_device(0)
            s = torch.cuda.Stream()
            for r in range(6):
                x = names[(i + r) % len(names)]
                if gp.count(graph, plans[x], stream=s) != want[x]:
                    bad.append((i, r, x))

        ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not bad
        graph.close()


@pytest.mark.parametrize("stride", [1, 2, 3, 64])
def test_iep_table_by_sample_stride(stride):
    """Samples dense enough for the table and samples past that rule, around a hub
    of 2,400 neighbors: the parts sum to the oracle's count, alone and in a batch."""
    k, e = P["house"]
    rng = np.random.default_rng(stride)
    n = 2500
    src = np.concatenate([np.zeros(2400, np.int64), rng.integers(0, n, 5000)])
    dst = np.concatenate([np.arange(1, 2401), rng.integers(0, n, 5000)])
    g = I.csr_from_edges(n, src, dst)
    want = O.count(g, k, e)
    graph = gp.Graph.from_csr(g, device=True)
    plan = gp.Plan(k, e, stats=graph.stats(), force_order=(0, 1, 2, 3, 4), force_restr=[(1, 0)], iep=True)
    assert plan.info().iep == 2 and plan.info().iep_div == 1
    assert sum(gp.count(graph, plan, root_stride=stride, root_offset=o) for o in range(stride)) == want
    batch = gp.Batch(graph, [plan])
    total = 0
    for o in range(stride):
        batch.set_sample(stride, o)
        total += batch.run()[0]
    assert total == want
    batch.close()
    graph.close()


def test_default_width_fits_the_workspace():
    """Two hubs over n leaves and a path of r leaf edges: r 4-cliques. Buffers
    of n ids for a block of 16-lane groups exceed the allocation-free call's
    workspace, those of 64-lane groups fit: a launch that names no width counts."""
    import torch
    n, r = 600_000, 1000
    leaf = np.arange(2, n + 2)
    src = np.concatenate([[0], np.zeros(n, np.int64), np.ones(n, np.int64), leaf[:r]])
    dst = np.concatenate([[1], leaf, leaf, leaf[1:r + 1]])
    graph = gp.Graph.from_csr(I.csr_from_edges(n + 2, src, dst), device=True)
    plan = gp.Plan(*P["4-clique"], stats=graph.stats())
    out = torch.zeros(2, dtype=torch.int64, device="cuda")
    with pytest.raises(gp.GpError):
        gp.count_noalloc(graph, plan, out, group=16)
    gp.count_noalloc(graph, plan, out)
    torch.cuda.synchronize()
    assert out.tolist() == [r, 0]
    assert gp.count(graph, plan) == r
    graph.close()


@pytest.mark.parametrize("n,m,hub", [(3, 3, 0), (12, 64, 0), (30, 65, 0), (40, 129, 0), (200, 800, 70), (600, 500, 599),
                                     (2000, 20000, 1500)])
def test_triangles_with_edges_sharing_a_walk(n, m, hub):
    """Triangle counts that walk 64 edges' lists as one: few edges, last
    windows of every length, lists with and without bitmaps, hubs whose lists
    pass one step of the walk, samples, and every configuration of the pattern."""
    rng = np.random.default_rng(m)
    src = np.concatenate([rng.integers(0, n, m), np.zeros(hub, np.int64)])
    dst = np.concatenate([rng.integers(0, n, m), np.arange(1, hub + 1)])
    g = I.csr_from_edges(n, src, dst)
    k, e = P["triangle"]
    want = O.count(g, k, e)
    for opts in (dict(), dict(hub_min_degree=200), dict(hub_bitmaps="dense"), dict(hub_bitmaps="none")):
        graph = gp.Graph.from_csr(g, device=True, **opts)
        for order in itertools.permutations(range(3)):
            for fs in range(gp.Plan(k, e).info().n_sets):
                plan = gp.Plan(k, e, stats=graph.stats(), force_order=order, force_set=fs)
                assert gp.count(graph, plan) == want, (opts, order, fs)
                assert gp.count_traffic(graph, plan)[0] == want
                assert sum(gp.count(graph, plan, root_stride=3, root_offset=o) for o in range(3)) == want
                assert gp.count(graph, plan, group=32) == want
        graph.close()
