"""GPU parity of the tiled asynchronous loop (AUTO on mesh-like graphs): every
result equals the CPU oracle's Dijkstra bit for bit (tolerance 0)."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


def lattice(dims, moves, wlo, whi, seed, wtype=gg.W_U32, perm=False, drop=0.0, extra=()):
    """A lattice graph: arcs along `moves` (both ways), seeded weights, ids
    permuted on request, a share of the arcs dropped (directed then)."""
    rng = np.random.default_rng(seed)
    n = int(np.prod(dims))
    at = np.stack(np.unravel_index(np.arange(n), dims), 1)
    src, dst = [], []
    for mv in moves:
        for sgn in (1, -1):
            to = at + sgn * np.asarray(mv)
            ok = ((to >= 0) & (to < np.asarray(dims))).all(1) & (rng.random(n) >= drop)
            src.append(np.flatnonzero(ok))
            dst.append(np.ravel_multi_index(tuple(to[ok].T), dims))
    src, dst = np.concatenate(src + [np.array([a for a, _ in extra], np.int64)]), \
        np.concatenate(dst + [np.array([b for _, b in extra], np.int64)])
    if perm:
        p = rng.permutation(n)
        src, dst = p[src], p[dst]
    if wtype == gg.W_F32:
        w = (rng.random(len(src)) * whi).astype(np.float32).view(np.uint32)
    else:
        w = rng.integers(wlo, whi, len(src), endpoint=True).astype(np.uint32)
    order = np.argsort(src, kind="stable")
    ro = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(src, minlength=n), out=ro[1:])
    return gg.CSR(n=n, ro=ro, col=dst[order].astype(np.int32), w=w[order], wtype=wtype, name="lattice")


FOUR = [(0, 1), (1, 0)]
EIGHT = FOUR + [(1, 1), (1, -1)]
SIX3D = [(0, 0, 1), (0, 1, 0), (1, 0, 0)]
hub = [(2100, int(x)) for x in np.random.default_rng(1).integers(0, 9000, 40)]

CASES = {
    "one tile, exactly full": lambda: lattice((64, 56), FOUR, 1, 100, 1, gg.W_F32),
    "one vertex past a tile": lambda: lattice((1, 3585), FOUR, 1, 100, 2, gg.W_F32),
    "a full square of places": lambda: lattice((64, 64), FOUR, 1, 100, 13, gg.W_F32),
    "two tiles, ragged": lambda: lattice((83, 79), FOUR, 1, 100, 3, gg.W_F32),
    "permuted ids": lambda: lattice((300, 211), FOUR, 1, 1000, 4, perm=True),
    "zero weights": lambda: lattice((150, 150), FOUR, 0, 2, 5),
    "directed, unreachable parts": lambda: lattice((140, 130), FOUR, 1, 9, 6, drop=0.35),
    "eight neighbours": lambda: lattice((120, 110), EIGHT, 1, 255, 7),
    "eight neighbours, binary32": lambda: lattice((101, 97), EIGHT, 1, 1, 8, gg.W_F32, perm=True),
    "three dimensions": lambda: lattice((24, 25, 26), SIX3D, 1, 255, 9),
    "a hub past the arc columns": lambda: lattice((100, 100), FOUR, 1, 50, 10, extra=hub),
    "uint32 saturation": lambda: lattice((90, 90), FOUR, 1 << 25, 1 << 27, 11),
    "binary32 overflow": lambda: lattice((90, 90), FOUR, 1, 1e37, 12, gg.W_F32),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_tiled_matches_oracle(name):
    g = CASES[name]()
    srcs = [0, g.n - 1, g.n // 2 + 7]
    with gr.Graph.from_csr(g) as G:
        for s in srcs:
            print("tiled %s n=%d m=%d src=%d" % (name, g.n, g.m, s), file=sys.stderr, flush=True)
            for rep in range(2):  # the second query reuses pool memory
                d = torch.full((g.n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
                st = gr.gr_sssp_ex(G.handle, s, d, barrier_timeout_us=2000000)
                torch.cuda.synchronize()
                # the route: one phase, an initialisation and one persistent launch
                assert st["loop"] == gr.GR_LOOP_ASYNC and st["iterations"] == 1 and st["launches"] == 2
                np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, s))


def test_tiled_not_taken():
    # no locality (a random graph of several tiles), and requests that name a
    # round-based schedule: the loops they had
    g = gg.uniform(30000, 60000, 3, 4, symmetric=True)
    with gr.Graph.from_csr(g) as G:
        d = torch.empty(g.n, dtype=torch.int32, device="cuda")
        st = gr.gr_sssp_ex(G.handle, 5, d)
        torch.cuda.synchronize()
        assert st["frontier_sum"] > 0 and not (st["loop"] == gr.GR_LOOP_ASYNC and st["layout"] == 2)
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, 5))
    g = gg.grid(300, wseed=4)
    with gr.Graph.from_csr(g) as G:
        d = torch.empty(g.n, dtype=torch.int32, device="cuda")
        for kw in (dict(filter=3), dict(local_hops=2), dict(delta=100), dict(direction=gr.GR_DIR_ALTERNATE),
                   dict(relax_filter=2), dict(layout=gr.GR_LAYOUT_PLAIN)):
            st = gr.gr_sssp_ex(G.handle, 5, d, **kw)
            torch.cuda.synchronize()
            assert st["loop"] == gr.GR_LOOP_QUEUED, kw
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, 5))
        with pytest.raises(gr.GrError) as ei:
            gr.gr_sssp_ex(G.handle, 5, d, max_iters=3)
        assert ei.value.status == gr.GR_ERR_ITER_LIMIT


def test_tiled_tuned():
    g = gg.grid(200, wseed=5)
    with gr.Graph.from_csr(g) as G:
        r = G.tune([0, 777], reps=1)
        assert 0 < r["best_ms"] <= r["default_ms"]
        d = torch.empty(g.n, dtype=torch.int32, device="cuda")
        gr.gr_sssp(G.handle, 9, d)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, 9))


def test_tiled_bfs_and_batch():
    g = lattice((300, 230), EIGHT, 1, 255, 21, perm=True)  # 69,000 vertices: breadth-first search too
    srcs = [0, 68999, 5, 5, 31000]
    with gr.Graph.from_csr(g) as G:
        d = torch.empty(g.n, dtype=torch.int32, device="cuda")
        st = gr.gr_bfs_ex(G.handle, 7, d)
        torch.cuda.synchronize()
        assert st["loop"] == gr.GR_LOOP_ASYNC
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.bfs(g, 7))
        rows = torch.full((len(srcs), g.n), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        st = gr.gr_sssp_batch_ex(G.handle, srcs, rows)
        torch.cuda.synchronize()
        assert st["replays"] == 0 and st["rounds"] == 1
        for s, row in zip(srcs, rows.cpu().numpy().view(np.uint32)):
            np.testing.assert_array_equal(row, oracle.dijkstra(g, s))
    g = gg.grid(90, wseed=8)
    with gr.Graph.from_csr(g) as G:  # the most queries of one launch
        srcs = gg.pick_sources(g, 5, 64)
        rows = torch.full((64, g.n), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        gr.gr_sssp_batch(G.handle, srcs, rows)
        torch.cuda.synchronize()
        for s, row in zip(srcs, rows.cpu().numpy().view(np.uint32)):
            np.testing.assert_array_equal(row, oracle.dijkstra(g, int(s)))


def test_tiled_multi_and_server():
    # both slot counts and weight types over tiles, beside graphs that have none
    graphs = [gg.grid(110, wseed=3), lattice((100, 90), EIGHT, 1, 9, 4), lattice((95, 101), FOUR, 1, 5, 5, gg.W_F32),
              gg.rmat(11, 8, gseed=1, pseed=2, wseed=3), gg.grid(30, wseed=6),
              lattice((2, 5000), FOUR, 1, 70000, 7, extra=[])]
    Gs = [gr.Graph.from_csr(g) for g in graphs]
    try:
        qs = [(i % len(graphs), (977 * i) % graphs[i % len(graphs)].n) for i in range(30)]
        want = [oracle.dijkstra(graphs[i], s) for i, s in qs]
        outs = [torch.full((graphs[i].n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda") for i, _ in qs]
        st = gr.gr_sssp_multi([Gs[i].handle for i, _ in qs], [s for _, s in qs], outs)
        torch.cuda.synchronize()
        for (i, s), o, w in zip(qs, outs, want):
            np.testing.assert_array_equal(o.cpu().numpy().view(np.uint32), w, err_msg=str((i, s)))
        assert len(st["iterations"]) == len(qs) and max(st["iterations"]) <= st["rounds"]
        for destroy_first in (False, True):  # queries still queued when the server goes are run first
            outs = [torch.full((graphs[i].n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda") for i, _ in qs]
            torch.cuda.synchronize()
            server = gr.gr_server_create(1 << 30)
            ids = [gr.gr_server_add_graph(server, G.handle) for G in Gs]
            tickets = [gr.gr_serve_submit(server, ids[i], s, o) for (i, s), o in zip(qs, outs)]
            if not destroy_first:
                for t, (i, s) in zip(tickets, qs):
                    r = None
                    while r is None:
                        r = gr.gr_serve_poll(server, t)
                    assert r["status"] == gr.GR_OK and r["src"] == s and r["batch_size"] >= 1
            gr.gr_server_destroy(server)
            torch.cuda.synchronize()
            for (i, s), o, w in zip(qs, outs, want):
                np.testing.assert_array_equal(o.cpu().numpy().view(np.uint32), w, err_msg=str((i, s)))
    finally:
        for G in Gs:
            G.close()
