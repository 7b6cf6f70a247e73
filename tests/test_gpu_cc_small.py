"""Components at the edges of their splits: as many remaining vertices and
arcs as one workgroup takes and one more, a remainder that overflows the
workgroups' buffers, a largest component of high ids only, iterations past
one launch's share, vertex counts around a bitmap word, labels that are not
16-byte aligned."""
import numpy as np
import pytest

import oracle
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw, trees

pytestmark = pytest.mark.gpu


def _big_and_rest(rest_vertices, rest_arcs, shift=0, tail=3):
    """`shift` isolated vertices, `rest_vertices` in pairs and one path (an odd
    count ends in a path of three) with `rest_arcs` arcs in all (made up by
    repeated edges), then a star that holds most of the graph."""
    src, dst, v = [], [], shift
    while rest_vertices - (v - shift) >= 2 and rest_vertices - (v - shift) != 3:
        src.append(v), dst.append(v + 1)
        v += 2
    if rest_vertices - (v - shift) == 3:
        src += [v, v + 1]
        dst += [v + 1, v + 2]
        v += 3
    while 2 * len(src) < rest_arcs:
        src.append(shift), dst.append(shift + 1)
    hub = v + 2 * 6000
    src += [hub] * (2 * 6000)
    dst += list(range(v, v + 2 * 6000))
    src += [hub] * 60000
    dst += list(range(v, v + 60000))
    n = max(hub, v + 60000) + 1 + tail
    return gg.from_edges(n, src, dst, drop_loops=False, dedup=False, name="big_and_rest")


def _two(a, b, n_extra=0):
    rows = [np.repeat(np.arange(x.n), x.degrees()) for x in (a, b)]
    return gg.from_edges(a.n + b.n + n_extra, np.concatenate([rows[0], rows[1] + a.n]),
                         np.concatenate([a.cols, b.cols + a.n]), name="two")


def _path(n):
    return gg.from_edges(n, list(range(n - 1)), list(range(1, n)), name="path")


GRAPHS = {
    "rest_none": lambda: _big_and_rest(0, 0),
    "rest_4095": lambda: _big_and_rest(4095, 0),
    "rest_4096": lambda: _big_and_rest(4096, 0, shift=63),
    "rest_4097": lambda: _big_and_rest(4097, 0, shift=64),
    "arcs_32768": lambda: _big_and_rest(4000, 32768, shift=1),
    "arcs_32770": lambda: _big_and_rest(4000, 32770, shift=700),
    "high_ids": lambda: _big_and_rest(10, 0, shift=70001),
    "iterations": lambda: _two(_path(4001), gg.rmat(13, 16, seed=81)),
    "remainder_overflows": lambda: _two(gg.erdos_renyi(300007, 1200000, seed=82), gg.erdos_renyi(250013, 900000, seed=83)),
    "rmat12_ragged": lambda: _two(gg.rmat(12, 8, seed=84), _path(1), n_extra=12),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_components_edges(name):
    import torch

    g = GRAPHS[name]()
    G = gsw.Graph.from_csr(g.offs, g.cols)
    want, count = oracle.components(g.offs, g.cols)
    for policy in ("switch", "push", "pull"):
        for bfs_first in (True, False):
            buf = torch.full((g.n + 1,), 7, dtype=torch.int32, device="cuda")
            for out in (buf[:g.n], buf[1:]):  # aligned, and off by one element
                lab, nc, tr = gsw.components(G, policy=policy, bfs_first=bfs_first, device=True, out=out,
                                             tree=trees.load_default())
                assert nc == count and np.array_equal(out.cpu().numpy(), want), (policy, bfs_first)
                it = tr[1:] if bfs_first else tr
                assert [t["iteration"] for t in tr] == list(range(len(tr)))
                if it:
                    assert it[-1]["changed"] == 0 and all(r["changed"] > 0 for r in it[:-1])
    G.close()
