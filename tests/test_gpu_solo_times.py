"""The cost per level that training rows get for single-workgroup levels: only
on levels that every push kernel runs that way."""
import numpy as np
import pytest

from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw, train

pytestmark = pytest.mark.gpu


def test_hub_level_keeps_its_own_times():
    """A path of 40 vertices into a hub of 12000 leaves: push_vertex runs the
    hub's level in one workgroup, push_edge spreads it over the grid."""
    hub, leaves = 40, 12000
    src = np.concatenate([np.arange(hub), np.full(leaves, hub)])
    dst = np.concatenate([np.arange(1, hub + 1), np.arange(hub + 1, hub + 1 + leaves)])
    make = lambda: gg.from_edges(hub + 1 + leaves, src, dst, name="path_hub")  # noqa: E731
    depth = hub + 2
    rows = dict(graph=np.array(["path_hub"] * depth), source=np.zeros(depth, dtype=np.int64), level=np.arange(depth))
    out = train.solo_times([("path_hub", make, None)], rows, log=lambda *a: None)
    assert np.isnan(out[hub]) and np.isfinite(out[:hub]).sum() >= 30  # (a grid launch between two of these)
    g = make()
    G = gsw.Graph.from_csr(g.offs, g.cols)
    for kernel, solo in ((gsw.PUSH_VERTEX, True), (gsw.PUSH_EDGE, False)):
        tr = gsw.bfs(G, [0], policy="fixed", kernel=kernel)[2]
        assert bool(tr[hub].flags & 4) == solo
    G.close()
