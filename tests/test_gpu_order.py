"""GPU parity of the weight-ordered loop (AUTO on graphs without locality):
every result equals the CPU oracle's Dijkstra bit for bit (tolerance 0)."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


def stars(degrees, n, seed, wlo=0, whi=60, wtype=gg.W_U32, both=True):
    """Vertex i has degrees[i] arcs to random heads (parallel arcs and
    self-loops among them), mirrored on request, and a sparse ring."""
    rng = np.random.default_rng(seed)
    src = np.concatenate([np.full(d, i) for i, d in enumerate(degrees)] + [np.arange(0, n, 3)])
    dst = np.concatenate([rng.integers(0, n, d) for d in degrees] + [(np.arange(0, n, 3) + 1) % n])
    if both:
        src, dst = np.concatenate([src, dst]), np.concatenate([dst, src])
    if wtype == gg.W_F32:
        w = (rng.random(len(src)) * whi).astype(np.float32).view(np.uint32)
    else:
        w = rng.integers(wlo, whi, len(src), endpoint=True).astype(np.uint32)
    order = np.argsort(src, kind="stable")
    ro = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(src, minlength=n), out=ro[1:])
    return gg.CSR(n=n, ro=ro, col=dst[order].astype(np.int32), w=w[order], wtype=wtype, name="stars")


EDGE = [1, 2, 3, 8, 9, 10, 63, 64, 65, 66, 127, 128, 129, 1022, 1023, 1024, 1025, 1026, 2048, 2049, 5000]

CASES = {
    "skewed": lambda: gg.rmat(15, 16, gseed=1, pseed=2, wseed=3),
    "skewed, binary32": lambda: gg.rmat(14, 16, gseed=4, pseed=5, wseed=6, wtype=gg.W_F32),
    "skewed, thin": lambda: gg.rmat(17, 3, gseed=7, pseed=8, wseed=9, whi=100000),
    "rows at the sort's edges": lambda: stars(EDGE * 3, 30011, 10),
    "rows at the sort's edges, directed, binary32": lambda: stars(EDGE * 3, 20000, 11, wtype=gg.W_F32, both=False),
    "zero weights": lambda: stars([400] * 50, 15000, 12, wlo=0, whi=1),
    "uint32 saturation": lambda: stars([300] * 60, 20000, 13, wlo=1 << 30, whi=0xFFFFFFFE),
    "binary32 overflow": lambda: stars([300] * 60, 20000, 14, whi=3e38, wtype=gg.W_F32),
    "bounded degree, no locality": lambda: gg.uniform(90001, 300000, 15, 16, symmetric=True),
    "bounded degree, directed": lambda: gg.uniform(70000, 400000, 17, 18, wlo=0, whi=3),
    "a chain with a hub (pushes only)": lambda: gg.from_arcs(
        30000, [(i, i + 1, 1 + i % 7) for i in range(2000)] + [(5, 20000 + i, i) for i in range(80)]),
    "a bitmap's last word": lambda: stars([200] * 40, 65 * 512 + 1, 19),
}


def query(G, n, s, **kw):
    d = torch.full((n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    st = gr.gr_sssp_ex(G.handle, int(s), d, **kw)
    torch.cuda.synchronize()
    return d.cpu().numpy().view(np.uint32), st


@pytest.mark.parametrize("name", sorted(CASES))
def test_ordered_matches_oracle(name):
    g = CASES[name]()
    with gr.Graph.from_csr(g) as G:
        for s in [0, g.n - 1] + [int(x) for x in gg.pick_sources(g, 3, 3)]:
            print("ordered %s n=%d m=%d src=%d" % (name, g.n, g.m, s), file=sys.stderr, flush=True)
            want = oracle.dijkstra(g, s)
            for rep in range(2):  # the second query enqueues the first one's rounds
                got, st = query(G, g.n, s)
                np.testing.assert_array_equal(got, want)
                # the route: a launch per round after the first one, no filter
                assert st["loop"] == gr.GR_LOOP_QUEUED and st["launches"] >= st["iterations"] + 1


@pytest.mark.parametrize("n", [(3 << 18) - 1, 3 << 18, (3 << 18) + 1])
def test_ordered_large(n):
    # from 786,432 vertices on, what a row needs is loaded ahead
    for wtype in (gg.W_U32, gg.W_F32):
        g = stars(EDGE * 200, n, 41, wtype=wtype)
        s = int(gg.pick_sources(g, 3, 1)[0])
        print("ordered n=%d m=%d src=%d" % (g.n, g.m, s), file=sys.stderr, flush=True)
        want = oracle.dijkstra(g, s)
        with gr.Graph.from_csr(g) as G:
            for rep in range(2):
                got, st = query(G, g.n, s)
                np.testing.assert_array_equal(got, want)
                assert st["loop"] == gr.GR_LOOP_QUEUED and 0 < st["arcs_pulled"]


def test_ordered_not_taken():
    g = gg.rmat(13, 16, gseed=21, pseed=22, wseed=23)
    s = int(gg.pick_sources(g, 3, 1)[0])
    want = oracle.dijkstra(g, s)
    with gr.Graph.from_csr(g) as G:
        for kw in (dict(direction=gr.GR_DIR_PUSH), dict(direction=gr.GR_DIR_PULL), dict(filter=1), dict(delta=50),
                   dict(relax_filter=1), dict(alpha_x16=8), dict(loop=gr.GR_LOOP_HOST)):
            got, st = query(G, g.n, s, **kw)
            np.testing.assert_array_equal(got, want, err_msg=str(kw))
            assert st["edges_pushed"] > g.m or st["arcs_pulled"] % g.m == 0, kw
        with pytest.raises(gr.GrError) as ei:
            query(G, g.n, s, max_iters=1)
        assert ei.value.status == gr.GR_ERR_ITER_LIMIT
        ordered = query(G, g.n, s)[1]
        assert 0 < ordered["arcs_pulled"] < g.m
    with gr.Graph.from_csr(g, flags=gr.GR_NO_PULL) as G:
        got, st = query(G, g.n, s)
        np.testing.assert_array_equal(got, want)
        assert st["arcs_pulled"] == 0


def test_ordered_tuned(tmp_path, monkeypatch):
    monkeypatch.setenv("GR_TUNE_CACHE", str(tmp_path / "t.jsonl"))
    g = gg.rmat(14, 8, gseed=24, pseed=25, wseed=26, wtype=gg.W_F32)
    srcs = gg.pick_sources(g, 3, 2)
    want = oracle.dijkstra(g, int(srcs[0]))
    stats = []
    for cached in (0, 1):  # what the cache says is what ran
        with gr.Graph.from_csr(g) as G:
            assert G.tune(srcs, reps=1)["from_cache"] == cached
            got, st = query(G, g.n, srcs[0])
            np.testing.assert_array_equal(got, want)
            stats.append((st["loop"], st["layout"], st["arcs_pulled"] > 0))
    assert stats[0] == stats[1]


def test_ordered_multi_and_server():
    graphs = [gg.rmat(14, 16, gseed=31, pseed=32, wseed=33), gg.rmat(13, 8, gseed=34, pseed=35, wseed=36, wtype=gg.W_F32),
              gg.uniform(70000, 300000, 37, 38), gg.grid(190, 39),
              gg.from_arcs(300, [(i, i + 1, 1) for i in range(299)])]  # (the last two run other loops)
    Gs = [gr.Graph.from_csr(g) for g in graphs]
    qs = [(i % len(graphs), int(s)) for i, g in enumerate(graphs) for s in list(gg.pick_sources(g, 3, 3)) + [g.n - 1]]
    want = [oracle.dijkstra(graphs[i], s) for i, s in qs]

    def rows():
        return [torch.full((graphs[i].n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda") for i, _ in qs]

    try:
        outs = rows()
        st = gr.gr_sssp_multi([Gs[i].handle for i, _ in qs], [s for _, s in qs], outs)
        torch.cuda.synchronize()
        for (i, s), o, w, it in zip(qs, outs, want, st["iterations"]):
            np.testing.assert_array_equal(o.cpu().numpy().view(np.uint32), w, err_msg=graphs[i].name)
            assert (it > 0) == bool(graphs[i].ro[s + 1] > graphs[i].ro[s])
        for destroy_first in (False, True):
            outs = rows()
            torch.cuda.synchronize()
            server = gr.gr_server_create(1 << 30)
            ids = [gr.gr_server_add_graph(server, G.handle) for G in Gs]
            tickets = [gr.gr_serve_submit(server, ids[i], s, o) for (i, s), o in zip(qs, outs)]
            if not destroy_first:
                for t in tickets:
                    while gr.gr_serve_poll(server, t) is None:
                        pass
            gr.gr_server_destroy(server)
            torch.cuda.synchronize()
            for o, w in zip(outs, want):
                np.testing.assert_array_equal(o.cpu().numpy().view(np.uint32), w)
    finally:
        for G in Gs:
            G.close()


@pytest.mark.parametrize("k", [2, 17, 64])
@pytest.mark.parametrize("name", sorted(CASES))
def test_ordered_batch(name, k):
    g = CASES[name]()
    # repeated sources, and one without arcs where the graph has it
    srcs = np.asarray(([0, g.n - 1] + [int(x) for x in gg.pick_sources(g, 3, 29)] * 3)[:k], np.int32)
    print("ordered batch %s n=%d m=%d k=%d" % (name, g.n, g.m, k), file=sys.stderr, flush=True)
    want = {int(s): oracle.dijkstra(g, int(s)) for s in set(srcs.tolist())}
    with gr.Graph.from_csr(g) as G:
        d = torch.empty(k, g.n, dtype=torch.int32, device="cuda")
        for rep in range(2):
            d.fill_(0x5A5A5A5A)
            st = gr.gr_sssp_batch_ex(G.handle, srcs, d)
            torch.cuda.synchronize()
            got = d.cpu().numpy().view(np.uint32)
            for i, s in enumerate(srcs):
                np.testing.assert_array_equal(got[i], want[int(s)], err_msg="row %d, source %d" % (i, s))
        arcs = int(np.diff(g.ro)[srcs].sum())  # (sources without arcs alone: no rounds)
        assert st["replays"] >= 1 and (st["rounds"] > 0) == (arcs > 0) and st["source_relaxations"] >= min(arcs, st["rounds"])
