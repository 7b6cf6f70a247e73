"""Canonical parents at the row lengths where the kernel changes its split
(lane, quarter wave, windows of a long row, more windows than their array
holds), on ascending and shuffled rows, against the smallest neighbour one level up."""
import numpy as np
import pytest

import oracle
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu


def _expect(offs, cols, level):
    n = offs.shape[0] - 1
    origin = np.repeat(np.arange(n), np.diff(offs))
    up = (level[cols] > 0) & (level[origin] == level[cols] - 1)
    want = np.full(n, np.iinfo(np.int32).max, dtype=np.int64)
    np.minimum.at(want, cols[up], origin[up])
    want[level < 0] = -1
    want[level == 0] = np.flatnonzero(level == 0)
    return want.astype(np.int32)


def _check(offs, cols, sources, flags=0):
    G = gsw.Graph.from_csr(offs, cols, flags=flags)
    lv, pa, _ = gsw.bfs(G, sources, policy="fixed", kernel=gsw.PUSH_EDGE, canonical_parents=True)
    for i, s in enumerate(sources):
        want = oracle.levels(offs, cols, int(s))
        assert np.array_equal(lv[i], want)
        assert np.array_equal(pa[i], _expect(offs, cols, want)), (i, int(s))


@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("deg", [1, 16, 17, 128, 129, 1023, 1024, 1025, 2048, 2049, 5000])
def test_row_length_edges(deg, shuffled):
    # two hubs of the given degree that share their leaves, joined to a root:
    # the hubs' parents come from the end of their rows, the leaves' from both
    rng = np.random.default_rng(deg)
    n = deg + 4
    hubs = (n - 2, 1)
    leaves = np.setdiff1d(np.arange(n), [*hubs, n - 1, 0])[: max(deg - 1, 0)]
    a = np.concatenate([np.full(leaves.size, h) for h in hubs] + [[n - 1, n - 1]]).astype(np.int64)
    b = np.concatenate([leaves, leaves, hubs]).astype(np.int64)
    key = np.unique(np.concatenate([a * n + b, b * n + a]))
    src, cols = key // n, (key % n).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int64)
    if shuffled:
        for v in range(n):
            rng.shuffle(cols[offs[v]:offs[v + 1]])
    sources = [n - 1] + ([int(leaves[-1])] if leaves.size else [])
    _check(offs, cols, sources)


@pytest.mark.parametrize("repeats", [1000, 4000, 20000])
def test_more_windows_than_room(repeats):
    # six vertices leave room for 48 windows of 1024 arcs; the rows of the
    # larger two need up to 280
    n = 6
    pairs = [(0, 1), (0, 2), (1, 3), (2, 3), (1, 4), (2, 4), (3, 5)]
    offs, cols = [0], []
    for v in range(n):
        row = [b if a == v else a for a, b in pairs if v in (a, b)]
        cols += row * repeats
        offs.append(len(cols))
    _check(np.array(offs, dtype=np.int64), np.array(cols, dtype=np.int32), [0, 5, 3])
