"""The tiled loop's bound on a wait is held against the query's progress: while
tiles run, workgroups without work wait for as long as it takes."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


@pytest.mark.parametrize("wtype", [gg.W_U32, gg.W_F32])
def test_a_path_longer_than_the_bound(wtype):
    # 56 tiles of a path run one or two at a time, 0.2 us or so per vertex: the
    # query takes ten times the bound and more, most workgroups never have work
    n = 200000
    w = np.arange(n - 1) % 7 + 1
    w = w.astype(np.float32).view(np.uint32) if wtype == gg.W_F32 else w.astype(np.uint32)
    ro = np.minimum(np.arange(n + 1), n - 1).astype(np.int32)
    g = gg.CSR(n=n, ro=ro, col=np.arange(1, n, dtype=np.int32), w=w, wtype=wtype, name="path")
    want = oracle.dijkstra(g, 0)
    with gr.Graph.from_csr(g) as G:
        for us in (2000, 1000):
            print("path of %d, bound %d us" % (n, us), file=sys.stderr, flush=True)
            d = torch.full((n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            st = gr.gr_sssp_ex(G.handle, 0, d, barrier_timeout_us=us, timing=1)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), want)
            assert st["loop"] == gr.GR_LOOP_ASYNC and st["launches"] == 2 and st["push_us"] > 2 * us


@pytest.mark.parametrize("back", [0, 1])
def test_arcs_and_expansions_of_a_path(back):
    # every vertex is improved once, so it is expanded once, over its own arcs
    # alone: the next one's, and with back the one it came from
    n = 9001
    i = np.arange(n - 1)
    g = gg.from_arcs(n, sorted([(int(a), int(a) + 1, 1.5) for a in i] + [(int(a) + 1, int(a), 2.5) for a in i] * back),
                     wtype=gg.W_F32)
    with gr.Graph.from_csr(g) as G:
        d = torch.full((n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        st = gr.gr_sssp_ex(G.handle, 0, d)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, 0))
        assert st["loop"] == gr.GR_LOOP_ASYNC and st["launches"] == 2
        assert st["frontier_sum"] == n and st["edges_pushed"] == g.m
