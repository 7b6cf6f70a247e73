"""Bottom-up levels at the edges of their splits: rows whose only frontier
neighbour is their last arc, of every length around the head copy, the arcs
that lanes and lane groups take and the part the whole wavefront finishes;
one to eight visited words a wavefront; few and many unresolved rows."""
import numpy as np
import pytest

import oracle
from oracle import checks
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu

LENGTHS = [1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 20, 21, 24, 31, 33, 64, 65, 255, 256, 257, 260, 261, 319, 320, 321, 512,
           513, 1000]


def _last_arc(copies, dead):
    """Source 0 -> f_i -> t_i, where t_i also has in-arcs from LENGTHS[i] - 1
    unreachable vertices of smaller id; `copies` of every length."""
    src, dst = [], []
    t0 = 1 + dead
    nt = copies * len(LENGTHS)
    f0 = t0 + nt
    for i in range(nt):
        k = LENGTHS[i % len(LENGTHS)]
        src.extend([0, f0 + i]), dst.extend([f0 + i, t0 + i])
        src.extend(range(1, k)), dst.extend([t0 + i] * (k - 1))
    return gg.from_edges(f0 + nt, src, dst, symmetrize=False, name="last_arc")


GRAPHS = {
    "last_arc": lambda: _last_arc(1, 1000),
    "last_arc_many": lambda: _last_arc(40, 1000),
    "rmat13": lambda: gg.rmat(13, 16, seed=71),
    "er_ragged": lambda: gg.erdos_renyi(9973, 30000, seed=72),
    "star": lambda: gg.from_edges(3001, [0] * 3000, list(range(1, 3001)), name="star"),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_pull_rows(name):
    g = GRAPHS[name]()
    G = gsw.Graph.from_csr(g.offs, g.cols)
    directed = name.startswith("last_arc")
    srcs = [0] if directed or name == "star" else [int(s) for s in gg.pick_sources(g, 2, 73)]
    if name == "star":
        srcs.append(3000)
    refs = [oracle.levels(g.offs, g.cols, s) for s in srcs]
    # launches of so few workgroups that a wavefront takes 1, 2, 4 or 8 words and several rounds
    for workgroups in (0, 1, 3, 6, 11, 20):
        lv, pa, tr = gsw.bfs(G, srcs, policy="fixed", kernel=gsw.PULL_BITMAP, max_workgroups=workgroups)
        assert all(t.kernel == gsw.PULL_BITMAP for t in tr)
        for i, s in enumerate(srcs):
            assert np.array_equal(lv[i], refs[i])
            (checks.check_bfs_directed if directed else checks.check_bfs)(g.offs, g.cols, s, lv[i], pa[i])
    G.close()


@pytest.mark.parametrize("n,children", [(262144, 1024), (262144, 1025), (262080, 1023), (70001, 273), (70001, 274),
                                        (4194304, 5000), (4194305, 5000), (4300007, 8192), (4300007, 8193)])
def test_pull_small_frontiers(n, children):
    """Frontiers on both sides of those a bottom-up level sums up in LDS, with
    one bit per 64 vertices and per 128; ids up to the last one."""
    rng = np.random.default_rng(n + children)
    ids = np.concatenate([[n - 1, 0, 63, 64], rng.permutation(np.arange(65, n - 1))])
    hub, kids, leaves = ids[0], ids[1:1 + children], ids[1 + children:1 + 4 * children]
    src = np.concatenate([np.full(children, hub), rng.choice(kids, leaves.size), rng.choice(kids, leaves.size)])
    dst = np.concatenate([kids, leaves, leaves])
    g = gg.from_edges(n, src, dst, name="two_levels")
    G = gsw.Graph.from_csr(g.offs, g.cols, flags=gsw.ASSUME_SYMMETRIC | gsw.TRUSTED)
    for s in (int(hub), int(leaves[0])):
        ref = oracle.levels(g.offs, g.cols, s)
        lv, pa, tr = gsw.bfs(G, [s], policy="fixed", kernel=gsw.PULL_BITMAP)
        assert np.array_equal(lv[0], ref)
        checks.check_bfs(g.offs, g.cols, s, lv[0], pa[0])
        assert [t.n_frontier for t in tr] == np.bincount(ref[ref >= 0]).tolist()
    G.close()
