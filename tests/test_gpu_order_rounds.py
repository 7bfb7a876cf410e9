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
