"""The workloads whose speed this library is held to.

Every case is one call (or one round of served queries) through the public
entry points on graphs that stay resident, as a routing, network-analysis or
graph-serving program keeps them.  The graph families are the ones of the
benchmark: 4-neighbour meshes, road-like meshes with a few long shortcuts,
R-MAT graphs (skewed degrees) and uniformly random graphs, with uint32 or
binary32 weights.  Graphs are generated on the GPU from the seed alone.

A case is a dict:
  op       sssp | bfs | noalloc | batch (k sources, one graph) | multi (k
           queries over a set of graphs) | serve (k queries through a server)
  family   mesh | road | rmat | uniform, or "mixed" for multi / serve
  size     mesh, road: rows and cols; rmat: scale, ef; uniform: n, deg
  wt       u32 | f32, whi: uint32 weights are U[1, whi], binary32 U(0, 1]
  k        queries of batch, multi and serve; graphs: resident graphs of
           multi and serve
"""
import math
import time

import numpy as np
import torch

import paper_2212_08200_amd as gr

RMAT_A, RMAT_B, RMAT_C = 0.57, 0.19, 0.19


def listed():
    return [
        # One route on a small map tile: the smallest call, where latency is everything.
        dict(name="mesh64", op="sssp", family="mesh", rows=64, cols=64, wt="u32", whi=100),
        # A mid-size, ragged map with measured (binary32) lengths: too large for one compute unit.
        dict(name="mesh173x229_f32", op="sssp", family="mesh", rows=173, cols=229, wt="f32", whi=0),
        # The largest mesh of the serving set, queried alone.
        dict(name="mesh1024", op="sssp", family="mesh", rows=1024, cols=1024, wt="u32", whi=255),
        # A road network with long-distance links.
        dict(name="road2048", op="sssp", family="road", rows=2048, cols=2048, wt="u32", whi=1000),
        # The high-diameter stress case.
        dict(name="mesh2048", op="sssp", family="mesh", rows=2048, cols=2048, wt="u32", whi=1000),
        # A small skewed graph (a social neighbourhood): launches count.
        dict(name="rmat15", op="sssp", family="rmat", scale=15, ef=16, wt="u32", whi=255),
        # A mid-size skewed graph with binary32 weights.
        dict(name="rmat20_f32", op="sssp", family="rmat", scale=20, ef=16, wt="f32", whi=0),
        # The headline graph.
        dict(name="rmat22", op="sssp", family="rmat", scale=22, ef=16, wt="u32", whi=255),
        # Hop counts on the headline graph.
        dict(name="rmat22_bfs", op="bfs", family="rmat", scale=22, ef=16, wt="u32", whi=255),
        # Landmark tables: distances from many sources of one graph at once.
        dict(name="rmat20_batch64", op="batch", family="rmat", scale=20, ef=16, wt="u32", whi=255, k=64),
        # One query on each of several resident graphs in one call.
        dict(name="multi24", op="multi", family="mixed", graphs=12, k=24, wt="u32", whi=255),
        # A burst of requests to the query server over the resident graphs.
        dict(name="serve48", op="serve", family="mixed", graphs=12, k=48, wt="u32", whi=255),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choices(["sssp", "bfs", "noalloc", "batch", "multi", "serve"], [12, 3, 1, 3, 1, 1])[0]
    if op in ("multi", "serve"):
        return dict(op=op, family="mixed", graphs=rng.randint(3, 12), k=rng.randint(3, 48), wt="u32",
                    whi=rng.choice([100, 255, 1000]))
    family = rng.choices(["mesh", "road", "rmat", "uniform"], [4, 3, 4, 2])[0]
    wt = rng.choice(["u32", "u32", "f32"])
    c = dict(op=op, family=family, wt=wt, whi=rng.choice([100, 255, 1000]) if wt == "u32" else 0)
    many = op == "batch"
    if many:
        c["k"] = rng.randint(2, 64)
    if family in ("mesh", "road"):
        top = 96 if many else 2048
        low = 16 if family == "mesh" else 64
        c["rows"] = log_int(low, top)
        c["cols"] = min(top, max(low, int(c["rows"] * math.exp(rng.uniform(-0.7, 0.7)))))
    elif family == "rmat":
        c["scale"] = rng.randint(10, 19 if many else 22)
        c["ef"] = rng.randint(4, 16)
    else:
        c["n"] = log_int(1000, 250_000 if many else 2_000_000)
        c["deg"] = rng.randint(2, 24)
    return c


# ---- graphs ------------------------------------------------------------------


def _mixed(case):
    """The resident graphs of multi and serve: R-MAT of scale 14 to 18 and
    meshes of side 256 to 1024, taking turns."""
    sides = (256, 512, 768, 1024)
    out = []
    for i in range(case["graphs"]):
        if i % 2 == 0:
            out.append(dict(family="rmat", scale=14 + (i // 2) % 5, ef=16, wt=case["wt"], whi=case["whi"]))
        else:
            s = sides[(i // 2) % 4]
            out.append(dict(family="mesh", rows=s, cols=s, wt=case["wt"], whi=case["whi"]))
    return out


def _mix64(x):
    """A 64-bit finalizer (xor-shift, multiply) on int64 tensors."""
    for mul, sh in ((-49064778989728563, 33), (-4265267296055464877, 29)):
        x = (x ^ ((x >> sh) & ((1 << (64 - sh)) - 1))) * mul
    return x ^ ((x >> 32) & 0xFFFFFFFF)


def _weights(h, case):
    """Weights of arcs from 64-bit hashes: int32 tensor of the weight bits."""
    if case["wt"] == "f32":
        return (((h >> 40) & 0xFFFFFF).add_(1).to(torch.float32) * 2.0 ** -24).view(torch.int32)
    return (((h >> 33) & 0x7FFFFFFF) % case["whi"] + 1).to(torch.int32)


def _csr(n, key, seed, case, mirrored):
    """CSR of the sorted arc keys (tail * n + head)."""
    src, dst = key // n, (key % n)
    pair = torch.minimum(src, dst) * n + torch.maximum(src, dst) if mirrored else key
    w = _weights(_mix64(pair + (int(seed) * 2654435761 + 12345) % (1 << 52)), case)
    ro = torch.zeros(n + 1, dtype=torch.int32, device=key.device)
    ro[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0).to(torch.int32)
    return n, ro, dst.to(torch.int32), w


def _graph(case, seed):
    """(n, row offsets, heads, weight bits) on the GPU."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 7919 + 17)
    fam = case["family"]
    if fam in ("mesh", "road"):
        r, c = case["rows"], case["cols"]
        n = r * c
        v = torch.arange(n, dtype=torch.int64, device=dev)
        col = v % c
        key = torch.stack([v * n + v - c, v * n + v - 1, v * n + v + 1, v * n + v + c], 1)
        ok = torch.stack([v >= c, col > 0, col < c - 1, v < n - c], 1)
        key = key[ok]
        if fam == "road":
            a = torch.randint(n, (n // 1000, 2), generator=g, device=dev)
            a = a[a[:, 0] != a[:, 1]]
            key = torch.unique(torch.cat([key, a[:, 0] * n + a[:, 1], a[:, 1] * n + a[:, 0]]))
        return _csr(n, key, seed, case, False)
    if fam == "rmat":
        n = 1 << case["scale"]
        e = n * case["ef"]
        u = torch.zeros(e, dtype=torch.int64, device=dev)
        v = torch.zeros(e, dtype=torch.int64, device=dev)
        for _ in range(case["scale"]):
            x = torch.rand(e, generator=g, device=dev)
            u.mul_(2).add_(x >= RMAT_A + RMAT_B)
            v.mul_(2).add_(((x >= RMAT_A) & (x < RMAT_A + RMAT_B)) | (x >= RMAT_A + RMAT_B + RMAT_C))
        perm = torch.randperm(n, generator=g, device=dev)
        u, v = perm[u], perm[v]
    else:
        n = case["n"]
        e = max(1, n * case["deg"] // 2)
        u = torch.randint(n, (e,), generator=g, device=dev)
        v = torch.randint(n, (e,), generator=g, device=dev)
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    del u, v, keep
    return _csr(n, key, seed, case, True)


def _sources(ro, k, seed):
    """k sources drawn among the vertices with arcs."""
    live = torch.nonzero(ro[1:] > ro[:-1]).flatten()
    pick = np.random.RandomState((int(seed) * 31 + 7) % (1 << 31)).randint(0, max(1, live.numel()), k)
    return [int(s) for s in live[torch.from_numpy(pick).to(live.device)].cpu()] if live.numel() else [0] * k


class _Resident:
    """Resident graphs, and the server over them if there is one."""

    def __init__(self, parts, wt, served):
        t = gr.GR_W_F32 if wt == "f32" else gr.GR_W_U32
        self.graphs = [gr.Graph(n, ro, col, w, t, flags=gr.GR_INPUT_DEVICE) for n, ro, col, w in parts]
        self.server = gr.gr_server_create(8 << 30) if served else None
        if served:
            self.ids = [gr.gr_server_add_graph(self.server, g.handle) for g in self.graphs]

    def __del__(self):
        if getattr(self, "server", None):
            gr.gr_server_destroy(self.server)
        self.server = None
        for g in getattr(self, "graphs", []):
            g.close()


def _inputs(case, seed):
    """The CSR parts and the (graph, source) queries of a case."""
    subs = _mixed(case) if case["family"] == "mixed" else [case]
    parts = [_graph(c, seed * 64 + i) for i, c in enumerate(subs)]
    k = case.get("k", 1)
    if len(subs) == 1:
        return parts, [(0, s) for s in _sources(parts[0][1], k, seed)]
    return parts, [(i % len(subs), _sources(parts[i % len(subs)][1], 1, seed + i)[0]) for i in range(k)]


def prepare(case, seed):
    parts, queries = _inputs(case, seed)
    torch.cuda.synchronize()
    res = _Resident(parts, case["wt"], case["op"] == "serve")
    dt = torch.float32 if case["wt"] == "f32" and case["op"] != "bfs" else torch.int32
    dev = torch.device("cuda")
    if case["op"] == "batch":
        dist = torch.empty(len(queries), parts[0][0], dtype=dt, device=dev)
    else:
        dist = [torch.empty(parts[i][0], dtype=dt, device=dev) for i, _ in queries]
    return dict(op=case["op"], res=res, queries=queries, dist=dist)


# ---- one pass ------------------------------------------------------------------


def run(state):
    op, res, queries, dist = state["op"], state["res"], state["queries"], state["dist"]
    if op == "batch":
        gr.gr_sssp_batch(res.graphs[0].handle, [s for _, s in queries], dist)
    elif op == "multi":
        gr.gr_sssp_multi([res.graphs[i].handle for i, _ in queries], [s for _, s in queries], dist)
    elif op == "serve":
        open_ = [gr.gr_serve_submit(res.server, res.ids[i], s, d) for (i, s), d in zip(queries, dist)]
        while open_:
            left = []
            for t in open_:
                r = gr.gr_serve_poll(res.server, t)
                if r is None:
                    left.append(t)
                elif r["status"] != gr.GR_OK:
                    raise RuntimeError("query failed: %s" % gr.gr_status_string(r["status"]))
            open_ = left
            if open_:
                time.sleep(20e-6)
    else:
        call = {"sssp": gr.gr_sssp, "bfs": gr.gr_bfs, "noalloc": gr.gr_sssp_noalloc}[op]
        call(res.graphs[0].handle, queries[0][1], dist[0])
    return dist


# ---- what a pass cannot do without ----------------------------------------------


def _size(c):
    """(vertices, arcs); the arcs of R-MAT graphs by their usual share of repeated pairs."""
    if c["family"] in ("mesh", "road"):
        n = c["rows"] * c["cols"]
        return n, 4 * n - 2 * (c["rows"] + c["cols"]) + (2 * (n // 1000) if c["family"] == "road" else 0)
    if c["family"] == "rmat":
        n = 1 << c["scale"]
        return n, int(2 * c["ef"] * n * (1 - 0.3 * 2.0 ** (-(c["scale"] - 10) / 4.4)))
    return c["n"], c["n"] * c["deg"]


def work(case):
    """Each arc (8 bytes; 4 for hop counts) and row offset of each graph queried read once, each
    distance written once; one addition for each arc and query."""
    subs = _mixed(case) if case["family"] == "mixed" else [case]
    k = case.get("k", 1)
    arc = 4 if case["op"] == "bfs" else 8
    b = f = 0
    for i, c in enumerate(subs):
        n, m = _size(c)
        q = k if len(subs) == 1 else (k - i + len(subs) - 1) // len(subs)
        if q > 0:
            b += arc * m + 4 * (n + 1) + 4 * n * q
            f += m * q
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """Bellman-Ford in 64 bits over all arcs of the graph."""
    subs = _mixed(case) if case["family"] == "mixed" else [case]
    k = case.get("k", 1)
    cost = 0.0
    for i, c in enumerate(subs):
        n, m = _size(c)
        rounds = 2 * (c["rows"] + c["cols"]) if c["family"] in ("mesh", "road") else 40
        q = k if len(subs) == 1 else (k - i + len(subs) - 1) // len(subs)
        cost += max(q, 0) * rounds * (60e-6 + m / 8e9)
    if cost > 15:
        return None
    parts, queries = _inputs(case, seed)
    real = case["wt"] == "f32" and case["op"] != "bfs"
    tails = [torch.repeat_interleave(torch.arange(p[0], device=p[1].device), (p[1][1:] - p[1][:-1]).long())
             for p in parts]
    out = []
    for i, s in queries:
        n, ro, col, w = parts[i]
        head = col.long()
        if case["op"] == "bfs":
            step, inf = torch.ones_like(head), 1 << 40
        elif real:
            step, inf = w.view(torch.float32).double(), float(np.finfo(np.float32).max)
        else:
            step, inf = w.long(), 1 << 40
        d = torch.full((n,), inf, dtype=step.dtype, device=head.device)
        d[s] = 0
        for r in range(1, n + 2):
            old = d.clone()
            d.scatter_reduce_(0, head, torch.clamp(old[tails[i]] + step, max=inf), "amin")
            if r % 4 == 0 and torch.equal(old, d):
                break
        out.append(d if real else torch.where(d >= inf, -1, d).to(torch.int32))
    return torch.stack(out) if case["op"] == "batch" else out
