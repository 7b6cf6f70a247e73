"""Bottom-up levels over long rows beside each other: on both sides of the
numbers of rows and of the lengths up to which lanes walk their own, lane groups
share them and the whole wavefront takes one after another."""
import numpy as np
import pytest

import oracle
from oracle import checks
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [24, 25, 64, 65, 128])
def test_long_rows_beside_each_other(rows):
    """Source 0 -> f_i -> t_i, the t_i of one word or two; t_i's other in-arcs
    come first and from vertices that are never reached.  All rows of one
    length, then every second one short."""
    dead = 800
    t0 = (1 + dead + 63) // 64 * 64
    f0 = t0 + rows
    for length in (63, 64, 65, 68, 69, 255, 256, 257, 260, 261, 320, 321, 700):
        for short in (length, 5):
            lens = [length if i % 2 == 0 else short for i in range(rows)]
            src = [np.zeros(rows, int), np.arange(f0, f0 + rows)] + [np.arange(1, k) for k in lens]
            dst = [np.arange(f0, f0 + rows), np.arange(t0, t0 + rows)] + [np.full(k - 1, t0 + i) for i, k in enumerate(lens)]
            g = gg.from_edges(f0 + rows, np.concatenate(src), np.concatenate(dst), symmetrize=False, name="beside")
            G = gsw.Graph.from_csr(g.offs, g.cols)
            ref = oracle.levels(g.offs, g.cols, 0)
            assert (ref[t0:t0 + rows] == 2).all()
            for workgroups in (0, 1):  # a word a wavefront, and eight
                lv, pa, tr = gsw.bfs(G, [0], policy="fixed", kernel=gsw.PULL_BITMAP, max_workgroups=workgroups, solo=False)
                assert np.array_equal(lv[0], ref), (length, short)
                checks.check_bfs_directed(g.offs, g.cols, 0, lv[0], pa[0])
            G.close()


@pytest.mark.parametrize("n,degree", [(65000, 8), (66000, 8), (300000, 2), (300000, 8), (66000, -8)])
def test_summary_of_small_frontiers(n, degree):
    """All levels bottom-up, with fewer and more unvisited in-arcs than a
    summary of a small frontier is made for; degree < 0: directed."""
    rng = np.random.default_rng(n + degree)
    m = n * abs(degree)
    g = gg.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), symmetrize=degree > 0, name="random")
    G = gsw.Graph.from_csr(g.offs, g.cols)
    srcs = [int(s) for s in gg.pick_sources(g, 2, 3)]
    lv, pa, tr = gsw.bfs(G, srcs, policy="fixed", kernel=gsw.PULL_BITMAP)
    for i, s in enumerate(srcs):
        ref = oracle.levels(g.offs, g.cols, s)
        assert np.array_equal(lv[i], ref)
        (checks.check_bfs if degree > 0 else checks.check_bfs_directed)(g.offs, g.cols, s, lv[i], pa[i])
    G.close()
