"""Edges of the single-workgroup launches: frontiers of exactly as many
vertices as the workgroup holds and of one more, rows as long as the head
copy and one arc longer, more long rows than it sets aside, bitmaps on both
sides of what it keeps in LDS, searches past each level cap, trees on both
sides of what LDS holds -- levels equal the oracle, parents valid."""
import numpy as np
import pytest

import oracle
from oracle import checks
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu

SOLO = 4  # trace flag of a level run by a single-workgroup launch


def _diamonds(widest, tail, extra=0, legs=0, n=None):
    """A binary tree over `widest` vertices on its last level but one, mirrored
    back to one vertex, then a path of `tail`: `extra` chains of the same depth
    from the root widen every frontier by one each; each vertex of the widest
    level gets `legs` leaves."""
    src, dst, front, nv = [], [], [0], 1
    chains = [0] * extra
    while len(front) < widest:
        new = []
        for v in front:
            for _ in range(2):
                src.append(v), dst.append(nv), new.append(nv)
                nv += 1
        front = new
        for i in range(extra):
            src.append(chains[i]), dst.append(nv)
            chains[i] = nv
            nv += 1
    for v in front:
        for _ in range(legs):
            src.append(v), dst.append(nv)
            nv += 1
    while len(front) > 1:
        new = []
        for i in range(0, len(front), 2):
            src.extend(front[i:i + 2]), dst.extend([nv, nv]), new.append(nv)
            nv += 1
        front = new
    v = front[0]
    for _ in range(tail):
        src.append(v), dst.append(nv)
        v, nv = nv, nv + 1
    assert n is None or nv <= n
    return gg.from_edges(n or nv, src, dst, name="diamond")


def _wide_tree(depth):
    """A complete decision tree of 2^(depth+1) - 1 nodes over the frontier and
    discovered fractions whose leaves all name queue-driven kernels."""
    inner = 2 ** depth - 1
    nodes = 2 * inner + 1
    rng = np.random.default_rng(3)
    thr = np.where(np.arange(nodes) < inner, 10.0 ** rng.uniform(-5, 0, nodes), -2.0)
    value = np.zeros((nodes, 3))
    value[np.arange(nodes), rng.integers(0, 3, nodes)] = 2.0
    return gsw.Tree(dict(left=[2 * i + 1 if i < inner else -1 for i in range(nodes)],
                         right=[2 * i + 2 if i < inner else -1 for i in range(nodes)],
                         feature=[(21, 23)[i % 2] if i < inner else -2 for i in range(nodes)],
                         threshold=thr.tolist(), value=value.tolist(),
                         class_kernel=[gsw.PUSH_VERTEX, gsw.PUSH_WAVE8, gsw.PUSH_EDGE]))


SHAPES = {
    "frontier_2048": dict(widest=2048, tail=10),
    "frontier_2049": dict(widest=2048, tail=10, extra=1),
    "frontier_4096_and_back": dict(widest=4096, tail=10),
    "rows_of_4": dict(widest=256, tail=40, extra=2),
    "rows_of_5": dict(widest=256, tail=40, extra=3),
    "long_rows_512": dict(widest=512, tail=5, legs=10),
    "long_rows_1024": dict(widest=1024, tail=5, legs=10),
    "bitmap_small": dict(widest=64, tail=130, n=131072),
    "bitmap_small_passed": dict(widest=64, tail=130, n=131073),
    "bitmap_largest": dict(widest=64, tail=300, n=1048576),
    "bitmap_too_large": dict(widest=64, tail=300, n=1048577),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_solo_edges(name):
    g = _diamonds(**SHAPES[name])
    n = g.n
    ref = oracle.levels(g.offs, g.cols, 0)
    sizes = np.bincount(ref[ref >= 0])
    G = gsw.Graph.from_csr(g.offs, g.cols)
    for kw in (dict(policy="fixed", kernel=gsw.PUSH_VERTEX), dict(policy="tree", tree=_wide_tree(6)),
               dict(policy="tree", tree=_wide_tree(8)),
               dict(policy="schedule", schedule=np.array([gsw.PUSH_VERTEX] * 7 + [gsw.PUSH_WAVE8], dtype=np.int32))):
        for count_arcs in (False, True):
            lv, pa, tr = gsw.bfs(G, [0, 0], count_arcs=count_arcs, trace_cap=1024, **kw)
            for i in range(2):
                assert np.array_equal(lv[i], ref)
                checks.check_bfs(g.offs, g.cols, 0, lv[i], pa[i])
                rows = [t for t in tr if t.source_idx == i]
                assert [t.n_frontier for t in rows] == sizes.tolist()
                assert not any(t.flags & SOLO and t.n_frontier > 2048 for t in rows)
                if kw["policy"] == "fixed":
                    assert sum(1 for t in rows if t.flags & SOLO) >= 0.5 * len(rows)
    G.close()


@pytest.mark.parametrize("children,leaves", [(15, 127), (16, 127), (16, 128), (63, 129), (511, 2), (513, 2), (186, 10),
                                             (187, 10), (750, 10), (2047, 0), (2048, 0), (2049, 0), (4600, 0)])
def test_solo_start_of_a_search_at_its_arc_limit(children, leaves):
    """A hub's level and its children's, with arcs on both sides of what one
    workgroup takes uncounted by degree (2048)."""
    src, dst, nv = [], [], 1 + children
    for c in range(1, children + 1):
        src.append(0), dst.append(c)
        src.extend([c] * leaves), dst.extend(range(nv, nv + leaves))
        nv += leaves
    g = gg.from_edges(nv, src, dst, name="hub")
    G = gsw.Graph.from_csr(g.offs, g.cols)
    for s in (0, nv - 1):
        ref = oracle.levels(g.offs, g.cols, s)
        sizes = np.bincount(ref[ref >= 0])
        for kernel in (gsw.PUSH_VERTEX, gsw.PUSH_EDGE):
            for count_arcs in (False, True):
                lv, pa, tr = gsw.bfs(G, [s], policy="fixed", kernel=kernel, count_arcs=count_arcs)
                assert np.array_equal(lv[0], ref)
                checks.check_bfs(g.offs, g.cols, s, lv[0], pa[0])
                assert [t.n_frontier for t in tr] == sizes.tolist()
                assert not any(t.flags & SOLO and t.e_frontier > 8192 for t in tr)
    G.close()


def _tiny_graphs():
    path = gg.from_edges(2048, list(range(2047)), list(range(1, 2048)), name="path2048")
    hub = gg.from_edges(2048, [0] * 2047 + [1] * 2000, list(range(1, 2048)) + list(range(2, 2002)), name="hubs")
    ragged = gg.rmat(10, 14, seed=91)
    a = gg.rmat(10, 8, seed=92)
    rows = np.repeat(np.arange(a.n), a.degrees())
    keep = np.random.default_rng(5).random(a.nnz) < 0.6
    directed = gg.from_edges(a.n, rows[keep], a.cols[keep], symmetrize=False, name="dir")
    clique = gg.from_edges(181, np.repeat(np.arange(181), 181), np.tile(np.arange(181), 181), name="clique")  # 32580 arcs
    over = gg.from_edges(182, np.repeat(np.arange(182), 182), np.tile(np.arange(182), 182), name="over")  # 32942
    wide = gg.from_edges(2049, list(range(2048)), list(range(1, 2049)), name="path2049")
    lone = gg.from_edges(1, [], [], name="one")
    return {g.name if g.name != "rmat" else "rmat10": g for g in (path, hub, directed, clique, over, wide, lone)} | {
        "ragged": ragged}


@pytest.mark.parametrize("name", ["path2048", "hubs", "dir", "clique", "over", "path2049", "one", "ragged"])
def test_whole_graph_in_one_workgroup(name):
    """Graphs on both sides of what one workgroup searches to the end: every
    kernel it runs, bottom-up included, schedules that leave and come back."""
    g = _tiny_graphs()[name]
    G = gsw.Graph.from_csr(g.offs, g.cols, flags=gsw.WITH_ORIGIN)
    srcs = sorted({0, g.n // 2, g.n - 1})
    refs = [oracle.levels(g.offs, g.cols, s) for s in srcs]
    check = checks.check_bfs if G.symmetric else checks.check_bfs_directed
    scheds = [[gsw.PULL_BITMAP], [gsw.PUSH_VERTEX, gsw.PULL_BITMAP], [gsw.PULL_BITMAP, gsw.PUSH_EDGE] * 60,
              [gsw.PUSH_EDGE, gsw.VERTEX_SCAN, gsw.PULL_BITMAP, gsw.PUSH_WAVE8, gsw.REV_EDGE_SCAN] * 20 + [gsw.PULL_BITMAP]]
    for kw in [dict(policy="fixed", kernel=k) for k in (gsw.PULL_BITMAP, gsw.PUSH_EDGE,
                                                        gsw.kernel_id(gsw.PULL_BITMAP, gsw.COUNT_WAVE))] + \
              [dict(policy="schedule", schedule=np.array(s, dtype=np.int32)) for s in scheds] + \
              [dict(policy="tree", tree=_wide_tree(6))]:
        for extra in (dict(), dict(count_arcs=True), dict(time_levels=True)):
            lv, pa, tr = gsw.bfs(G, srcs, trace_cap=8192, **kw, **extra)
            lv0, _, tr0 = gsw.bfs(G, srcs, trace_cap=8192, solo=False, **kw, **extra)
            assert [(t.source_idx, t.level, t.kernel, t.flags & ~SOLO, t.n_frontier, t.discovered, t.n_next, t.e_frontier)
                    for t in tr] == [(t.source_idx, t.level, t.kernel, t.flags, t.n_frontier, t.discovered, t.n_next,
                                      t.e_frontier) for t in tr0]
            for i, s in enumerate(srcs):
                assert np.array_equal(lv[i], refs[i]) and np.array_equal(lv0[i], refs[i])
                check(g.offs, g.cols, s, lv[i], pa[i])
            if kw.get("kernel") == gsw.PULL_BITMAP and len(tr):
                assert all(bool(t.flags & SOLO) == (name not in ("over", "path2049")) for t in tr)
    G.close()


@pytest.mark.parametrize("arcs", [2048, 2049, 8192, 8193])
def test_solo_rows_that_a_level_kernel_leaves_to_one_workgroup(arcs):
    """A level of few long rows: counted arcs up to 8192 for the lane-per-row
    kernels, up to 2048 for push_edge; 16 rows and 17 at the next level."""
    for rows in (16, 17):
        src, dst = [0] * arcs, list(range(1, arcs + 1))
        nv = arcs + 1
        for c in range(1, rows + 1):  # below a second root: rows of 200 arcs
            src.append(nv), dst.append(nv + c)
        for c in range(1, rows + 1):
            src.extend([nv + c] * 200), dst.extend(range(nv + rows + 1 + 200 * c, nv + rows + 201 + 200 * c))
        n = nv + rows + 201 + 200 * rows + 20000  # (isolated vertices: the average degree stays low)
        g = gg.from_edges(n, src, dst, name="rows")
        G = gsw.Graph.from_csr(g.offs, g.cols)
        for s in (0, nv):
            ref = oracle.levels(g.offs, g.cols, s)
            for kernel in (gsw.PUSH_VERTEX, gsw.PUSH_WAVE16, gsw.PUSH_EDGE):
                lv, pa, tr = gsw.bfs(G, [s], policy="fixed", kernel=kernel, count_arcs=True)
                assert np.array_equal(lv[0], ref)
                checks.check_bfs(g.offs, g.cols, s, lv[0], pa[0])
                few = kernel != gsw.PUSH_EDGE
                for t in tr[:2]:
                    if t.n_frontier <= 17 and t.n_frontier * int(g.degrees().max()) > 8192:
                        limit = 8192 if few and t.n_frontier <= 16 else 2048
                        assert bool(t.flags & SOLO) == (t.e_frontier <= limit), (s, kernel, t)
        G.close()


@pytest.mark.parametrize("n", [200003, 1100003])
@pytest.mark.parametrize("lead", [20, 29, 30, 31, 32, 33, 60, 100])
def test_solo_frontiers_where_the_bitmap_moves(lead, n):
    """A path, then frontiers of 1, 2, 4 .. 4096 vertices and back, twice: they
    pass what a launch takes with the bitmap in global memory (1024) and in LDS
    (2048) before, while and after later launches hold it in LDS (from depth
    32, if it fits)."""
    src, dst, nv, at = [], [], 1, 0

    def path(k):
        nonlocal nv, at
        for _ in range(k):
            src.append(at), dst.append(nv)
            at, nv = nv, nv + 1

    for _ in range(2):
        path(lead)
        front = [at]
        while len(front) < 4096:
            new = list(range(nv, nv + 2 * len(front)))
            nv += 2 * len(front)
            src.extend(v for v in front for _ in range(2)), dst.extend(new)
            front = new
        while len(front) > 1:
            new = list(range(nv, nv + len(front) // 2))
            nv += len(new)
            src.extend(front), dst.extend(v for v in new for _ in range(2))
            front = new
        at = front[0]
    path(5)
    g = gg.from_edges(n, src, dst, name="bulges")
    G = gsw.Graph.from_csr(g.offs, g.cols)
    ref = oracle.levels(g.offs, g.cols, 0)
    for kw in (dict(policy="fixed", kernel=gsw.PUSH_VERTEX), dict(policy="fixed", kernel=gsw.PUSH_EDGE),
               dict(policy="tree", tree=_wide_tree(6))):
        for count_arcs in (False, True):
            lv, pa, tr = gsw.bfs(G, [0], trace_cap=4096, count_arcs=count_arcs, **kw)
            assert np.array_equal(lv[0], ref)
            checks.check_bfs(g.offs, g.cols, 0, lv[0], pa[0])
            assert [t.n_frontier for t in tr] == np.bincount(ref[ref >= 0]).tolist()
            limit = 2048 if n <= 1048576 else 1024
            assert not any(t.flags & SOLO and t.n_frontier > limit for t in tr)
            assert sum(1 for t in tr if t.flags & SOLO) >= 0.5 * len(tr)
    G.close()
