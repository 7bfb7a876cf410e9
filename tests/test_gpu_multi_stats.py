"""Statistics of gr_sssp_multi calls whose queries take several loops: rounds and
replays are of loops that ran."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


def multi(Gs, graphs, qs):
    outs = [torch.full((graphs[i].n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda") for i, _ in qs]
    st = gr.gr_sssp_multi([Gs[i].handle for i, _ in qs], [s for _, s in qs], outs)
    torch.cuda.synchronize()
    for (i, s), o in zip(qs, outs):
        np.testing.assert_array_equal(o.cpu().numpy().view(np.uint32), oracle.dijkstra(graphs[i], s), err_msg=str((i, s)))
    return st


def test_replays_are_of_chunks_that_ran():
    graphs = [gg.grid(60, wseed=3), gg.grid(150, wseed=4), gg.rmat(13, 16, gseed=5, pseed=6, wseed=7)]
    Gs = [gr.Graph.from_csr(g) for g in graphs]
    try:
        small = [(0, 0), (0, 1800)]
        print("multi statistics", file=sys.stderr, flush=True)
        alone = multi(Gs, graphs, small)  # the single-workgroup loop: a hop per round, no chunks
        assert alone["replays"] == 0 and alone["rounds"] >= 100
        tiles = multi(Gs, graphs, [(1, 0), (1, 77)])
        assert tiles["replays"] == 0 and tiles["rounds"] == 1
        # beside the tiles, in the session's rounds, which take several hops each
        for qs in (small + [(1, 0)], small + [(1, 9), (2, 3)]):
            st = multi(Gs, graphs, qs)
            assert 1 < st["rounds"] < alone["rounds"] // 2 and st["rounds"] == max(st["iterations"])
            assert st["rounds"] / 8 <= st["replays"] <= st["rounds"] // 8 + 6
    finally:
        for G in Gs:
            G.close()
