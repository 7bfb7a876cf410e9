"""GPU parity of the breadth-first pull that knows its level (the host-driven
loop's): a vertex's in-arcs are read a line of eight at a time until one comes
from the frontier.  Depths equal the CPU oracle's (tolerance 0)."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")

# in-degrees around a line of arcs, the four lines read first and the windows of the rest
EDGE = [1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 34, 40, 63, 64, 65, 255, 256, 257, 1055, 1056, 1057, 5000]


@pytest.mark.parametrize("where", ["first", "last", "none"])
def test_bfs_level_pull_rows(where):
    # row v has EDGE[i] in-arcs; the one from a reached vertex stands first or
    # last in it (in-arcs are ordered by tail), or there is none
    rows, far = 600, 6000  # tails 1000 ... are never reached
    deg = [EDGE[i % len(EDGE)] for i in range(rows)]
    hub = 0 if where == "first" else 1000 + far
    n = hub + 1 + rows if where != "first" else 1000 + far + rows
    base = n - rows
    arcs = [(hub, 1 + (i % 900), 1) for i in range(900)]
    for i, d in enumerate(deg):
        tails = list(range(1000, 1000 + d - (0 if where == "none" else 1)))
        arcs += [(u, base + i, 1) for u in tails] + ([] if where == "none" else [(hub, base + i, 1)])
    arcs.sort()
    g = gg.from_arcs(n, arcs)
    want = oracle.bfs(g, hub)
    assert int((want[base:] == 1).sum()) == (0 if where == "none" else rows)
    with gr.Graph.from_csr(g) as G:
        for kw in (dict(direction=gr.GR_DIR_PULL), dict(direction=gr.GR_DIR_ALTERNATE), dict()):
            for rf in (0, gr.GR_RELAX_BOUND):
                d = torch.full((n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
                print("level pull", where, kw, rf, file=sys.stderr, flush=True)
                gr.gr_bfs_ex(G.handle, hub, d, loop=gr.GR_LOOP_HOST, relax_filter=rf, **kw)
                torch.cuda.synchronize()
                np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), want)
