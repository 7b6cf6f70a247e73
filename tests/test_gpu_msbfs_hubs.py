"""Hub rows of a batch, looked up by one wave and in chunks, in one search: few
sources that go bottom-up by their own frontiers, together and one after
another, with many hubs in one word of the bitmap and the hubs' rows found or
walked in vain."""
import numpy as np
import pytest

import oracle
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu


def _graph():
    rng = np.random.default_rng(31)
    n = 60000
    src = np.concatenate([rng.integers(0, 40, 70000), rng.integers(0, n, 90000), [40, 41]])
    dst = np.concatenate([rng.integers(0, n, 70000), rng.integers(0, n, 90000), [3, n - 1]])
    return gg.from_edges(n, src, dst, name="hubs")


@pytest.mark.parametrize("sources", [1, 2, 3, 5, 64, 65])
def test_hub_rows(sources):
    g = _graph()
    assert (g.degrees()[:40] > 1024).all()
    G = gsw.Graph.from_csr(g.offs, g.cols)
    rng = np.random.default_rng(sources)
    for first in (0, 40, 50000):  # a hub, its neighbour, one like most
        srcs = np.concatenate([[first], rng.integers(0, g.n, sources - 1)]).astype(np.int32)
        ref, ok = oracle.msbfs_levels(g.offs, g.cols, srcs)
        assert ok
        for p in (None, 0.0001, 0.01, 0.3, 1e9):
            lv, _ = gsw.msbfs(G, srcs, push_to_pull=p)
            assert np.array_equal(lv, ref), (first, p)
    G.close()


def test_hub_rows_of_a_session():
    g = _graph()
    G = gsw.Graph.from_csr(g.offs, g.cols)
    ss = gsw.Session(G, 64)
    rng = np.random.default_rng(5)
    todo, slots = [int(v) for v in rng.integers(0, g.n, 24)], {}
    while todo or slots:
        for v in todo[:2]:  # two more at every level: young and old ones side by side
            slots[ss.admit(v)] = v
        todo = todo[2:]
        for k in ss.step(1)[0]:
            v = slots.pop(k)
            assert np.array_equal(ss.fetch(k), oracle.levels(g.offs, g.cols, v)), v
    ss.close()
    G.close()


@pytest.mark.parametrize("degree", [33, 40, 62, 66, 128, 129, 200])
def test_long_rows_in_one_word(degree):
    """Few to many rows beside each other that one lane, a quarter wave or a wave
    looks up, found early, late and not at all: a path of 90 vertices with leaves."""
    for beside in (1, 3, 15, 17, 31, 33, 64, 90):
        k = 90
        per = [degree - 2 if i % 64 < beside else 3 for i in range(k)]
        spine = np.arange(k)
        leaf = np.repeat(spine, per)
        g = gg.from_edges(k + leaf.size, np.concatenate([spine[:-1], leaf]),
                          np.concatenate([spine[1:], np.arange(k, k + leaf.size)]), name="caterpillar")
        G = gsw.Graph.from_csr(g.offs, g.cols)
        rng = np.random.default_rng(beside)
        for B in (1, 2, 40):
            srcs = rng.integers(0, g.n, B).astype(np.int32)
            ref, ok = oracle.msbfs_levels(g.offs, g.cols, srcs)
            assert ok
            for p in (None, 0.0001):
                lv, _ = gsw.msbfs(G, srcs, push_to_pull=p)
                assert np.array_equal(lv, ref), (beside, B, p)
        G.close()
