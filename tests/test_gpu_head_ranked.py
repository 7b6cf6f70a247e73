"""The ranked head copy (graphs of skewed degrees), seen through bottom-up
searches: a vertex's parent is the first of its row's four in-neighbours of
largest out-degree (among the first 256 arcs, an earlier arc first among equal
degrees) that is one level up, else the first such in row order.  Rows of
every length around the splits, equal degrees, repeated arcs, directed and
undirected."""
import numpy as np
import pytest

import oracle
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu

HEAD, SCAN = 4, 256


def _in_rows(g, symmetric):
    if symmetric:
        return g.offs, g.cols
    src = np.repeat(np.arange(g.n), g.degrees())
    order = np.argsort(g.cols, kind="stable")
    return np.concatenate([[0], np.cumsum(np.bincount(g.cols, minlength=g.n))]), src[order]


def _parents(g, symmetric, level, source):
    offs, cols = _in_rows(g, symmetric)
    deg = g.degrees()
    out = np.full(g.n, -1, dtype=np.int64)
    for v in np.flatnonzero(level > 0):
        row = cols[offs[v]:offs[v + 1]]
        first = row[:SCAN]
        head = first[np.lexsort((np.arange(first.size), -deg[first]))][:HEAD]
        for u in np.concatenate([head, row]):
            if level[u] == level[v] - 1:
                out[v] = u
                break
    out[source] = source
    return out


def _lengths():
    """Hubs and rows of many lengths: vertex i of the second part has LENS[i]
    neighbours among the hubs and the first part, most with equal degrees."""
    lens = [1, 2, 3, 4, 5, 6, 7, 8, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 258, 300, 511]
    rng = np.random.default_rng(7)
    src, dst, base = [], [], 600
    for i, k in enumerate(lens * 6):
        pick = rng.choice(600, size=k, replace=False)
        src += [base + i] * k
        dst += pick.tolist()
    for h in range(12):  # hubs 0..11
        leaves = rng.choice(np.arange(12, 600), size=500, replace=False)
        src += [h] * 500
        dst += leaves.tolist()
    return gg.from_edges(base + len(lens) * 6 + 3000, src, dst, name="lengths")


def _graph(name):
    if name == "lengths":
        return _lengths(), True
    if name == "repeats":
        a = gg.rmat(11, 40, seed=61)
        rows = np.repeat(np.arange(a.n), a.degrees())
        rep = np.random.default_rng(62).integers(0, rows.size, 9000)
        return gg.from_edges(a.n, np.concatenate([rows, rows[rep]]), np.concatenate([a.cols, a.cols[rep]]),
                             drop_loops=False, dedup=False, name="repeats"), True
    a = gg.rmat(13, 12, seed=63)
    if name == "rmat13":
        return a, True
    rows = np.repeat(np.arange(a.n), a.degrees())
    keep = np.random.default_rng(64).random(a.nnz) < 0.6
    return gg.from_edges(a.n, rows[keep], a.cols[keep], symmetrize=False, name="directed"), False


@pytest.mark.parametrize("name", ["lengths", "repeats", "rmat13", "directed"])
def test_bottom_up_parents_follow_the_ranked_head(name):
    g, symmetric = _graph(name)
    assert g.degrees().std() > g.nnz / g.n  # so the head is ranked
    G = gsw.Graph.from_csr(g.offs, g.cols)
    assert bool(G.symmetric) == symmetric
    for s in gg.pick_sources(g, 2, 65):
        want_lv = oracle.levels(g.offs, g.cols, int(s))
        want = _parents(g, symmetric, want_lv, int(s))
        lv, pa, _ = gsw.bfs(G, [int(s)], policy="fixed", kernel=gsw.PULL_BITMAP)
        assert np.array_equal(lv[0], want_lv)
        assert np.array_equal(pa[0], want)
    G.close()
