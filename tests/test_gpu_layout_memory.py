"""Graphs whose second layouts (tiles, in-arcs by weight) do not fit in memory
are created without them and run the loops that need none: every result equals
the CPU oracle's Dijkstra (tolerance 0)."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")

GRAPHS = {
    "tiles": lambda: gg.grid(300, wseed=3),
    "by weight": lambda: gg.rmat(13, 16, gseed=4, pseed=5, wseed=6),
    "by weight, directed": lambda: gg.uniform(70000, 300000, 7, 8, wtype=gg.W_F32),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_created_without_the_layout(name, monkeypatch):
    g = GRAPHS[name]()
    s = int(gg.pick_sources(g, 3, 1)[0])
    want = oracle.dijkstra(g, s)
    sizes, stats = [], []
    for limit in (None, "4096", "0"):
        if limit is not None:
            monkeypatch.setenv("GR_LAYOUT_LIMIT", limit)
        print("layout limit", limit, name, file=sys.stderr, flush=True)
        with gr.Graph.from_csr(g) as G:
            sizes.append(G.info()["dev_bytes"])
            d = torch.full((g.n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            stats.append(gr.gr_sssp_ex(G.handle, s, d))
            torch.cuda.synchronize()
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), want)
            rows = torch.full((9, g.n), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            gr.gr_sssp_batch(G.handle, [s] * 9, rows)
            torch.cuda.synchronize()
            for row in rows.cpu().numpy().view(np.uint32):
                np.testing.assert_array_equal(row, want)
    # no layout is held, and a loop that needs none ran
    assert sizes[0] > sizes[1] == sizes[2]
    for st in stats[1:]:
        assert st["loop"] in (gr.GR_LOOP_QUEUED, gr.GR_LOOP_HOST) and st["arcs_pulled"] == 0
