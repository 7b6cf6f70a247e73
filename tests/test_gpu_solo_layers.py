"""Layered graphs whose levels qualify for a single workgroup by their size
and are handed back for their arcs, or passed on, where the kernel takes two
launches a level (push_edge on more than 512 vertices): every search ends with
the oracle's levels, through gsw_bfs and gsw_bfs_noalloc."""
import numpy as np
import pytest

import oracle
from oracle import checks
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu

SOLO = 4  # trace flag of a level run by a single-workgroup launch


def _layers(sizes, per, n):
    """Layer by layer, every vertex has `per` neighbours in the layer before."""
    src, dst, first = [], [], 0
    for p, q in zip(sizes, sizes[1:]):
        c = np.arange(q)
        for k in range(per):
            # (one parent per child: they are shared out evenly)
            src.append(first + ((c * p // q if per == 1 else c + k) % p))
            dst.append(first + p + c)
        first += p
    return gg.from_edges(n, np.concatenate(src), np.concatenate(dst), name="layers")


PATH = [1] * 33
EDGE = [gsw.PUSH_EDGE]
MIXED = [gsw.PUSH_EDGE, gsw.PUSH_VERTEX, gsw.PUSH_EDGE, gsw.PULL_BITMAP, gsw.PUSH_EDGE, gsw.PUSH_EDGE,
         gsw.VERTEX_SCAN, gsw.PUSH_WAVE8]
WHOLE = [gsw.VERTEX_SCAN, gsw.PUSH_VERTEX, gsw.PUSH_EDGE, gsw.PUSH_EDGE, gsw.PUSH_VERTEX, gsw.PUSH_EDGE]
CASES = {
    "layers_of_512": ([1, 16, 200] + [512] * 8, 8, 30000),
    "layers_of_513": ([1, 16, 200] + [513] * 8, 8, 30000),
    "layers_of_800": ([1, 16, 200] + [800] * 8, 8, 30000),
    "layers_of_1024": ([1, 16, 200] + [1024] * 8, 8, 30000),
    "layers_of_1025": ([1, 16, 200] + [1025] * 8, 8, 30000),
    "layers_of_600_long_rows": ([1, 16, 200] + [600] * 8, 20, 30000),
    "tail": ([1, 16, 250, 3000, 20000, 950, 700, 300, 60, 4], 8, 200003),
    "tail_in_global_memory": ([1, 16, 250, 3000, 20000, 950, 700, 600, 60, 4], 8, 1100003),
    "deep_800": (PATH + [16, 200] + [800] * 8, 8, 200003),
    "deep_2048": (PATH + [16, 200] + [2048] * 8, 8, 200003),
    "deep_2049": (PATH + [16, 200] + [2049] * 8, 8, 200003),
    "bounded_rows": (PATH + [3, 9, 27, 81, 243, 729, 1500, 2049, 4096, 2048, 4096, 2048, 30, 5], 1, 200003),
    "whole_graph": ([1, 20, 700, 600, 600, 30], 4, 2000),
}


@pytest.mark.parametrize("name", list(CASES))
def test_levels_handed_back_where_one_takes_two_launches(name):
    import torch

    sizes, per, n = CASES[name]
    g = _layers(sizes, per, n)
    G = gsw.Graph.from_csr(g.offs, g.cols)
    ref = oracle.levels(g.offs, g.cols, 0)
    count = np.bincount(ref[ref >= 0])
    assert count.max() >= 512 and (per == 1 or count.tolist() == sizes)
    deg_max = int(g.degrees().max())
    for sched in (EDGE, MIXED, WHOLE):
        kw = dict(policy="fixed", kernel=sched[0]) if len(sched) == 1 else \
            dict(policy="schedule", schedule=np.array(sched * 12, dtype=np.int32))
        for count_arcs in (True, False):
            lv, pa, tr = gsw.bfs(G, [0, 0], trace_cap=1024, count_arcs=count_arcs, **kw)
            for i in range(2):
                assert np.array_equal(lv[i], ref)
                checks.check_bfs(g.offs, g.cols, 0, lv[i], pa[i])
                rows = [t for t in tr if t.source_idx == i]
                assert [t.n_frontier for t in rows] == count.tolist()
                for t in rows:
                    if count_arcs and t.flags & SOLO and name != "whole_graph":
                        bounded = t.n_frontier * deg_max <= 8192
                        few = t.n_frontier <= 16 and gsw.kernel_base(t.kernel) != gsw.PUSH_EDGE
                        assert t.e_frontier <= (8192 if bounded or few else 2048), t
        if n <= 1 << 19:
            out = torch.full((2, n), 9, dtype=torch.int32, device="cuda")
            gsw.bfs_noalloc(G, [0, 0], out, **kw)
            assert np.array_equal(out.cpu().numpy(), np.stack([ref, ref]))
    G.close()
