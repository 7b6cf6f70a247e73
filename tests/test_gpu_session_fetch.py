"""A session's fetch into device memory returns when the levels are in place,
whatever the row's length (one workgroup, several, several rounds), for a
reader on any stream; the slot's next query starts from a clean row, and
fetches into host memory give the same levels."""
import numpy as np
import pytest

import oracle
from paper_1708_01159_amd import graphgen as gg
from paper_1708_01159_amd import gsw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 1024, 1025, 4096, 4097, 8195, 1048576, 1048577, 2100001])
def test_fetch_lengths(n):
    import torch

    # a star whose last vertex hangs off a leaf: levels 0, 1, 2 or 0, 1, 2, 3
    leaves = np.arange(1, max(n - 1, 2), dtype=np.int64)
    src = np.concatenate([np.zeros(leaves.size, dtype=np.int64), [1] if n > 2 else []]).astype(np.int64)
    dst = np.concatenate([leaves, [n - 1] if n > 2 else []]).astype(np.int64)
    g = gg.from_edges(n, src, dst, name="star")
    G = gsw.Graph.from_csr(g.offs, g.cols)
    ss = gsw.Session(G, 3)
    other = torch.cuda.Stream()
    for rnd in range(3):
        srcs = [0, n - 1, min(rnd + 1, n - 1)]
        want = [oracle.levels(g.offs, g.cols, s) for s in srcs]
        slots = {ss.admit(s): i for i, s in enumerate(srcs)}
        out = torch.full((3, n), 77, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        host = np.full(n, 77, dtype=np.int32)
        while slots:
            fin, _ = ss.step(8)
            for k in fin:
                i = slots.pop(k)
                if i == 2 and rnd == 1:
                    ss.fetch(k, out=host)
                    assert np.array_equal(host, want[i])
                    continue
                ss.fetch(k, out=out[i])
                with torch.cuda.stream(other):
                    copy = out[i].clone()
                other.synchronize()
                assert np.array_equal(copy.cpu().numpy(), want[i]), (rnd, i)
    assert ss.info()["busy"] == 0
    assert ss.info()["dev_bytes"] == gsw.lib().gsw_session_bytes(G.handle, 3)
    ss.close()
    G.close()
