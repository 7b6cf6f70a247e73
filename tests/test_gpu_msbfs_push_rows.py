"""The batch's top-down pass over rows on both sides of every length at which
its split changes (own lane, quarter wave, wave, chunks), alone and several to
a 64-vertex word, for every share of a vertex's mask words that pushes: levels
equal the oracle's, on a directed graph and top-down on a symmetric one."""
import numpy as np
import pytest

import oracle
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 4, 5, 16, 31, 32, 33, 64, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 1300]


def _graph(directed, n):
    """Roots 0..., each with a row of one of the lengths; words of 64 ids hold
    one row that is not short, two, three, four, five or many."""
    rng = np.random.default_rng(17)
    src, dst, at = [], [], 0
    for many in (1, 2, 3, 4, 5, 20):
        for k in range(len(LENGTHS)):
            for i in range(many):
                r = (at // 64) * 64 + i * 3 if i else at
                length = LENGTHS[(k + 7 * i) % len(LENGTHS)]
                src.append(np.full(length, r % n))
                dst.append(rng.choice(n, length, replace=False))
            at += 64
    s, d = np.concatenate(src), np.concatenate(dst)
    keep = s != d
    return gg.from_edges(n, s[keep], d[keep], symmetrize=not directed, name="rows"), np.arange(0, at, 64) % n


@pytest.mark.parametrize("directed,n", [(True, 9001), (False, 9001), (True, 32768), (True, 32769)])
def test_push_rows_of_every_length(directed, n):
    g, roots = _graph(directed, n)
    G = gsw.Graph.from_csr(g.offs, g.cols)
    rng = np.random.default_rng(18)
    # one source, a few, all of a word, part of two, three and four words, all of 16
    for B in (1, 3, 64, 65, 128, 130, 200, 256, 300, 1024):
        srcs = np.concatenate([roots, rng.integers(0, g.n, 1024)])[:B].astype(np.int32)
        if B in (64, 128):  # all at one vertex: its words push together
            srcs[:] = roots[20]
        ref, ok = oracle.msbfs_levels(g.offs, g.cols, srcs)
        assert ok
        for bs in (128, 512):
            lv, _ = gsw.msbfs(G, srcs, push_to_pull=1e9, block_size=bs)
            assert np.array_equal(lv, ref), (B, bs)
    G.close()
