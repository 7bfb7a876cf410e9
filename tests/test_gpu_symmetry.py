"""Which graphs count as symmetric (their out-arcs serve the pull direction):
every row strictly ascending and every arc with its reverse of equal weight."""
import sys

import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
gr = pytest.importorskip("paper_2212_08200_amd")


def base():
    # degrees on both sides of a row that the whole wave reads (256), a hub,
    # equal degrees, a self-loop and rows without arcs
    rng = np.random.default_rng(5)
    pairs = {(0, v): 3 for v in range(1, 1400)} | {(1500, v): 4 for v in range(1, 257)} | {(1501, v): 5 for v in range(300, 555)}
    for _ in range(6000):
        u, v = sorted(int(x) for x in rng.integers(1, 1400, 2))
        pairs[(u, v)] = int(rng.integers(1, 99))
    arcs = {}
    for (u, v), w in pairs.items():
        arcs[(u, v)] = arcs[(v, u)] = w
    return arcs


def csr(arcs):
    return gg.from_arcs(1600, sorted((u, v, w) for (u, v), w in arcs.items()))


def drop(arcs, k):
    del arcs[k]


def weight(arcs, k):
    arcs[k] += 1


EDITS = {
    "none": None,
    "an arc out of the hub": lambda a: drop(a, (0, 77)),
    "an arc into the hub": lambda a: drop(a, (77, 0)),
    "two arcs, one each way": lambda a: (drop(a, (0, 77)), drop(a, (88, 0))),
    "two arcs between others, one each way": lambda a: (drop(a, (1500, 9)), drop(a, (310, 1501))),
    "a weight": lambda a: weight(a, (1501, 300)),
    "a weight of the lighter end": lambda a: weight(a, (300, 1501)),
}


@pytest.mark.parametrize("edit", sorted(EDITS))
def test_symmetry(edit):
    arcs = base()
    if EDITS[edit]:
        EDITS[edit](arcs)
    g = csr(arcs)
    print("symmetry", edit, g.n, g.m, file=sys.stderr, flush=True)
    with gr.Graph.from_csr(g) as G:
        assert G.info()["has_csc"] == (0 if edit == "none" else 1)


def test_symmetry_of_unordered_rows():
    arcs = sorted((u, v, w) for (u, v), w in base().items())
    # a parallel arc each way, and two arcs of a row exchanged
    for bad in (arcs + [(1, 0, 3), (0, 1, 3)], [arcs[1], arcs[0]] + arcs[2:]):
        with gr.Graph.from_csr(gg.from_arcs(1600, bad)) as G:
            assert G.info()["has_csc"] == 1
