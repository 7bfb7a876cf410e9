"""The query server's memory budget holds for queries on graphs that run over
tiles or weight-ordered arcs: as many run together as fit it.  Results equal the
CPU oracle's Dijkstra (tolerance 0)."""
import sys
import time

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


def serve(graphs, qs, budget, **cfg):
    """Submits all queries at once; returns their results."""
    Gs = [gr.Graph.from_csr(g) for g in graphs]
    outs = [torch.full((graphs[i].n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda") for i, _ in qs]
    torch.cuda.synchronize()
    server = gr.gr_server_create(budget, **cfg)
    try:
        ids = [gr.gr_server_add_graph(server, G.handle) for G in Gs]
        tickets = [gr.gr_serve_submit(server, ids[i], s, o) for (i, s), o in zip(qs, outs)]
        res, t0 = [None] * len(qs), time.time()
        while any(r is None for r in res):
            for k, t in enumerate(tickets):
                if res[k] is None:
                    res[k] = gr.gr_serve_poll(server, t)
            assert time.time() - t0 < 60, "served queries did not finish"
            time.sleep(0.0005)
    finally:
        gr.gr_server_destroy(server)
        for G in Gs:
            G.close()
    for (i, s), o, r in zip(qs, outs, res):
        assert r["status"] == gr.GR_OK
        np.testing.assert_array_equal(o.cpu().numpy().view(np.uint32), oracle.dijkstra(graphs[i], s), err_msg=str((i, s)))
    return res


def test_weight_ordered_queries_within_the_budget():
    g = gg.rmat(13, 16, gseed=1, pseed=2, wseed=3)
    qs = [(0, int(s)) for s in gg.pick_sources(g, 4, 24)]
    # a query takes its two queues of 2^14 entries of 8 bytes, and 22 KB more or less
    one = 2 * 16 * 1024 * 8
    for fit in (1, 2, 5):
        print("budget for", fit, file=sys.stderr, flush=True)
        res = serve([g], qs, fit * one + one // 2)
        assert max(r["batch_size"] for r in res) <= fit
    assert max(r["batch_size"] for r in serve([g], qs, 1 << 30)) > 5


def test_budget_below_an_own_launch():
    # the session's workspace fits (28 bytes per vertex), the loop's own does not
    g = gg.rmat(12, 16, gseed=1, pseed=2, wseed=3)
    qs = [(0, int(s)) for s in gg.pick_sources(g, 4, 12)]
    res = serve([g], qs, 150000)
    assert all(r["iterations"] >= 1 for r in res) and max(r["batch_size"] for r in res) == 1


def test_all_kinds_share_a_small_budget():
    graphs = [gg.grid(300, wseed=3), gg.rmat(13, 16, gseed=4, pseed=5, wseed=6), gg.uniform(40000, 120000, 7, 8),
              gg.rmat(12, 8, gseed=9, pseed=10, wseed=11, wtype=gg.W_F32), gg.grid(40, wseed=5)]
    qs = [(i % len(graphs), (977 * i) % graphs[i % len(graphs)].n) for i in range(70)]
    print("shared budget", file=sys.stderr, flush=True)
    serve(graphs, qs, 28 * 90000 + 4096, num_streams=2)
    serve(graphs, qs, 28 * 90000 + 4096, num_streams=1, max_batch=2)
