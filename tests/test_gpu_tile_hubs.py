"""GPU parity of the tiled loop on meshes with a few vertices of many arcs, which
go to the tiles' lists of other arcs: up to what such a list holds over tiles,
past it on the loops without.  Results equal the CPU oracle's (tolerance 0)."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


def hubs(rows, cols, degs, seed, wtype=gg.W_U32, back=True, near=False):
    """A mesh whose vertices degs' index * 997 have that many arcs more: to random
    vertices, or (near) to those that follow them."""
    n = rows * cols
    v = np.arange(n)
    src = np.concatenate([v[v % cols != cols - 1], v[: n - cols]])
    dst = np.concatenate([v[v % cols != cols - 1] + 1, v[cols:]])
    src, dst = np.concatenate([src, dst]), np.concatenate([dst, src])
    rng = np.random.default_rng(seed)
    for i, d in enumerate(degs):
        h = (i * 997 + 5) % n
        t = (h + 2 + np.arange(d)) % n if near else rng.integers(0, n, d)
        src, dst = np.concatenate([src, np.full(d, h)]), np.concatenate([dst, t])
        if back:
            src, dst = np.concatenate([src, t]), np.concatenate([dst, np.full(d, h)])
    key = np.unique(src[src != dst] * n + dst[src != dst])
    w = rng.random(len(key)).astype(np.float32).view(np.uint32) if wtype == gg.W_F32 else \
        rng.integers(1, 99, len(key)).astype(np.uint32)
    ro = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(key // n, minlength=n), out=ro[1:])
    return gg.CSR(n=n, ro=ro, col=(key % n).astype(np.int32), w=w, wtype=wtype, name="hubs")


# graph, whether it runs over tiles
HUBS = {
    "65 arcs": (lambda: hubs(270, 250, [61], 1), True),
    "17 arcs and more": (lambda: hubs(270, 250, [13, 14, 20, 40, 59, 60], 9), True),
    "a few, binary32": (lambda: hubs(240, 300, [70, 300, 1000], 2, wtype=gg.W_F32), True),
    "inside the tile": (lambda: hubs(300, 300, [1000], 3, near=True), True),
    "out only": (lambda: hubs(260, 280, [64, 500, 900], 4, back=False, wtype=gg.W_F32), True),
    "nearly the list": (lambda: hubs(400, 300, [2500], 5, back=False), True),
    "past the list": (lambda: hubs(400, 300, [3100], 6), False),
    "past the degree": (lambda: hubs(500, 400, [9000], 7), False),
    "too many": (lambda: hubs(200, 200, [200] * 60, 8), False),
}


@pytest.mark.parametrize("name", sorted(HUBS))
def test_meshes_with_hubs(name):
    make, tiled = HUBS[name]
    g = make()
    srcs = [0, 5, g.n - 1]
    with gr.Graph.from_csr(g) as G:
        d = torch.empty(g.n, dtype=torch.int32, device="cuda")
        for s in srcs:
            print("hubs", name, g.n, g.m, s, file=sys.stderr, flush=True)
            d.fill_(0x5A5A5A5A)
            st = gr.gr_sssp_ex(G.handle, s, d, barrier_timeout_us=2000000)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, s))
            assert (st["loop"] == gr.GR_LOOP_ASYNC) == tiled
        gr.gr_bfs(G.handle, 7, d)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.bfs(g, 7))
        rows = torch.full((9, g.n), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        gr.gr_sssp_batch(G.handle, srcs * 3, rows)
        torch.cuda.synchronize()
        for s, row in zip(srcs * 3, rows.cpu().numpy().view(np.uint32)):
            np.testing.assert_array_equal(row, oracle.dijkstra(g, s))


@pytest.mark.parametrize("n,deg", [(20000, 3), (60001, 3), (150000, 2), (300000, 4)])
def test_random_graphs_of_low_degree_have_no_tiles(n, deg, monkeypatch):
    # their cells are trees, with few arcs on the borders; only the worklist of
    # the asynchronous loop without tiles has a capacity to overflow
    monkeypatch.setenv("GR_ASYNC_LIST_CAP", "64")
    g = gg.uniform(n, n * deg // 2, 3, 4, symmetric=True)
    s = int(gg.pick_sources(g, 3, 1)[0])
    with gr.Graph.from_csr(g) as G:
        d = torch.full((g.n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        st = gr.gr_sssp_ex(G.handle, s, d)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, s))
        assert st["loop"] == gr.GR_LOOP_QUEUED if n > 65536 else st["iterations"] > 1


@pytest.mark.parametrize("side", [150, 700])
def test_meshes_have_tiles(side, monkeypatch):
    monkeypatch.setenv("GR_ASYNC_LIST_CAP", "64")
    g = gg.grid(side, wseed=4)
    with gr.Graph.from_csr(g) as G:
        d = torch.full((g.n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        st = gr.gr_sssp_ex(G.handle, 9, d)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, 9))
        assert st["loop"] == gr.GR_LOOP_ASYNC and st["iterations"] == 1
