"""Levels of a batch come from bit planes: every mask width, ragged vertex
counts around the output tiles, and levels on both sides of each digit that
brings a plane into use; rows at the lengths where a walk changes its split
(lane, quarter wave, group, wave, listed chunks).  Against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu


def _check(g, srcs, **kw):
    G = gsw.Graph.from_csr(g.offs, g.cols)
    lv, _ = gsw.msbfs(G, srcs, **kw)
    want, ok = oracle.msbfs_levels(g.offs, g.cols, srcs)
    assert ok and np.array_equal(lv, want)
    # the planes of a shallow search must not show through in the next one
    lv, _ = gsw.msbfs(G, srcs[::-1].copy(), **kw)
    assert np.array_equal(lv, want[::-1])
    G.close()


@pytest.mark.parametrize("n", [1, 2, 3, 5, 127, 129, 1021, 1024, 2047])
@pytest.mark.parametrize("nsrc", [1, 31, 33, 64, 65, 129, 257, 513, 577, 1023])
def test_widths_and_ragged_sizes(n, nsrc):
    g = gg.erdos_renyi(n, 2 * n, seed=n) if n > 1 else gg.from_edges(1, [], [])
    srcs = np.random.default_rng(nsrc).integers(0, n, nsrc).astype(np.int32)
    _check(g, srcs)


@pytest.mark.parametrize("depth", [1, 2, 3, 4, 7, 8, 9, 15, 16, 31, 32, 63, 64, 65, 127])
@pytest.mark.parametrize("p2p", [(0.07, 0.01), (0.0, 0.0)])
def test_levels_at_digit_boundaries(depth, p2p):
    # a path of depth arcs with a fan at its far end, sources at the near end
    n = depth + 40
    a = list(range(depth)) + [depth - 1] * 39
    b = list(range(1, depth + 1)) + list(range(depth + 1, n))
    g = gg.from_edges(n, a, b)
    _check(g, np.array([0, 0, min(1, depth - 1)], dtype=np.int32), push_to_pull=p2p[0], pull_to_push=p2p[1])


@pytest.mark.parametrize("nsrc", [3, 64, 100, 180, 300, 600])
@pytest.mark.parametrize("deg", [8, 9, 16, 17, 32, 33, 64, 65, 512, 513, 1024, 1025, 1300])
def test_row_lengths(deg, nsrc):
    # two hubs with the same leaves, joined to each other's far leaf by a tail
    # each: a hub's row is walked for sources that only its last arcs reach
    n = deg + 24
    leaves = np.arange(deg)
    a = np.concatenate([np.full(deg, deg), np.full(deg, deg + 1), np.arange(deg + 1, n - 1), [0]])
    b = np.concatenate([leaves, leaves[::-1], np.arange(deg + 2, n), [n - 1]])
    g = gg.from_edges(n, a, b)
    srcs = np.random.default_rng(deg + nsrc).integers(0, n, nsrc).astype(np.int32)
    srcs[:3] = (deg, n - 1, n // 2)
    for p2p in ((0.07, 0.01), (0.0, 0.0), (1e9, 1e9)):
        _check(g, srcs, push_to_pull=p2p[0], pull_to_push=p2p[1])
