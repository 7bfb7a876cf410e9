"""GPU parity of the weight-ordered loop's rounds on graphs that leave the usual
course of a query (a few pushes, then pulls to the end): wide frontiers of short
rows.  Results equal the CPU oracle's Dijkstra (tolerance 0)."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


def arcs(g):
    return np.repeat(np.arange(g.n), np.diff(g.ro)), g.col.astype(np.int64)


def both_ways(n, src, dst, seed, wtype=gg.W_U32, whi=255):
    """The pairs as arcs both ways, with seeded weights."""
    keep = src != dst
    key = np.unique(np.minimum(src, dst)[keep] * n + np.maximum(src, dst)[keep])
    rng = np.random.default_rng(seed)
    if wtype == gg.W_F32:
        w = (rng.random(len(key)) * whi).astype(np.float32).view(np.uint32)
    else:
        w = rng.integers(1, whi, len(key), endpoint=True).astype(np.uint32)
    a, b = key // n, key % n
    a, b, w = np.concatenate([a, b]), np.concatenate([b, a]), np.concatenate([w, w])
    order = np.lexsort((b, a))
    ro = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(a, minlength=n), out=ro[1:])
    return gg.CSR(n=n, ro=ro, col=b[order].astype(np.int32), w=w[order], wtype=wtype, name="rounds")


def spokes(side, hubs, deg, seed, **kw):
    """A mesh with hubs of deg arcs to random vertices."""
    g = gg.grid(side, seed)
    s, d = arcs(g)
    rng = np.random.default_rng(seed)
    h = rng.choice(g.n, hubs, replace=False)
    return both_ways(g.n, np.concatenate([s] + [np.full(deg, x) for x in h]),
                     np.concatenate([d, rng.integers(0, g.n, hubs * deg)]), seed, **kw)


# more queue entries than waves, of 4 arcs (and up to 256: a hub's), and just about as many
WIDE = {
    "short rows": lambda: spokes(300, 1, 5000, 1),
    "short rows, binary32": lambda: spokes(280, 1, 5000, 2, wtype=gg.W_F32),
    "hubs among them": lambda: spokes(300, 12, 4000, 3),
    "few": lambda: spokes(90, 1, 3500, 4, wtype=gg.W_F32),
}


@pytest.mark.parametrize("name", sorted(WIDE))
def test_wide_frontiers_of_short_rows(name):
    g = WIDE[name]()
    with gr.Graph.from_csr(g) as G:
        for s in [0, g.n - 1, g.n // 2]:
            print("wide", name, g.n, g.m, s, file=sys.stderr, flush=True)
            d = torch.full((g.n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            st = gr.gr_sssp_ex(G.handle, int(s), d)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), oracle.dijkstra(g, int(s)))
            assert st["loop"] == gr.GR_LOOP_QUEUED and st["iterations"] > st["pull_iterations"]


def joined(scale, length, seed, **kw):
    """Two R-MAT graphs joined by a path: the frontier grows, shrinks to one
    vertex and grows again."""
    a, b = gg.rmat(scale, 16, gseed=seed, pseed=2, wseed=3), gg.rmat(scale, 12, gseed=seed + 1, pseed=5, wseed=6)
    (sa, da), (sb, db), n = arcs(a), arcs(b), a.n + b.n + length
    path = np.concatenate([gg.pick_sources(a, 3, 1), np.arange(a.n + b.n, n), a.n + gg.pick_sources(b, 3, 1)]).astype(np.int64)
    return both_ways(n, np.concatenate([sa, sb + a.n, path[:-1]]), np.concatenate([da, db + a.n, path[1:]]), seed, **kw)


def tailed(scale, length, seed, **kw):
    g = gg.rmat(scale, 16, gseed=seed, pseed=2, wseed=3)
    s, d = arcs(g)
    path = np.concatenate([gg.pick_sources(g, 3, 1), np.arange(g.n, g.n + length)]).astype(np.int64)
    return both_ways(g.n + length, np.concatenate([s, path[:-1]]), np.concatenate([d, path[1:]]), seed, **kw)


AGAIN = {  # graph, rounds that a path alone takes
    "joined": (lambda: joined(15, 300, 1), 300),
    "joined, binary32": (lambda: joined(14, 200, 5, wtype=gg.W_F32), 200),
    "joined, zero weights": (lambda: joined(14, 200, 7, whi=1), 200),
    "joined, large": (lambda: joined(19, 40, 9), 40),
    "a tail of a large graph": (lambda: tailed(20, 300, 11, wtype=gg.W_F32), 300),
}


@pytest.mark.parametrize("name", sorted(AGAIN))
def test_pushes_again_after_pulls(name):
    make, path = AGAIN[name]
    g = make()
    with gr.Graph.from_csr(g) as G:
        for s in [int(x) for x in gg.pick_sources(g, 5, 2)]:
            want = oracle.dijkstra(g, s)
            for rep in range(2):
                print("again", name, g.n, g.m, s, file=sys.stderr, flush=True)
                d = torch.full((g.n,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
                st = gr.gr_sssp_ex(G.handle, s, d)
                torch.cuda.synchronize()
                np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), want)
                # it pulled, and most rounds of the path pushed
                assert st["pull_iterations"] > 0
                assert st["iterations"] - st["pull_iterations"] > path // 2


@pytest.mark.parametrize("name", sorted(AGAIN))
def test_batch_pushes_again_after_pulls(name):
    g = AGAIN[name][0]()
    srcs = np.asarray(list(gg.pick_sources(g, 5, 9)) + [g.n - 1, 0], np.int32)  # (one on the path)
    with gr.Graph.from_csr(g) as G:
        rows = torch.empty(len(srcs), g.n, dtype=torch.int32, device="cuda")
        for rep in range(2):
            print("batch again", name, g.n, g.m, file=sys.stderr, flush=True)
            rows.fill_(0x5A5A5A5A)
            st = gr.gr_sssp_batch_ex(G.handle, srcs, rows)
            torch.cuda.synchronize()
            got = rows.cpu().numpy().view(np.uint32)
            for i in (0, 4, 9, 10):
                np.testing.assert_array_equal(got[i], oracle.dijkstra(g, int(srcs[i])), err_msg=str(srcs[i]))
            # the arcs read: at most all of them in each of the fifteen or so
            # rounds that either end's growth takes, not in those of the path
            assert st["rounds"] > AGAIN[name][1] and st["edges_pushed"] < 30 * g.m
