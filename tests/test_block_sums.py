"""Block-wide accumulators of the kernels: a word in LDS that one thread clears
and others then add to needs a barrier between the two on every path, which no
result shows reliably when it is missing.  Read from the sources: after the
statement that clears such words, a barrier comes before the next branch, loop
or use of one of them."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2212_08200_amd", "csrc")
CLEAR = re.compile(r"if \((?:t|threadIdx\.x)(?: == 0| < \w+)\)\s*(\{[^{}]*\}|[^;{}]*;)")


def kernels(text):
    """(name, body) of every kernel, comments taken out."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\s*\(", text):
        i = text.index("{", m.end())
        depth, j = 0, i
        while True:
            depth += {"{": 1, "}": -1}.get(text[j], 0)
            j += 1
            if depth == 0:
                break
        yield m.group(1), text[i:j]


def unordered(body):
    """Accumulators (words of LDS that are added to with an atomic) whose first
    clearing no barrier follows in time."""
    words = {w for d in re.findall(r"__shared__([^;]*);", body) for w in re.findall(r"\b(s[A-Z]\w*)", d)}
    sums = {w for w in words if re.search(r"\b(?:atomicAdd|atomicMin|atomicMax|atomicOr)\(&%s\b" % w, body)}
    bad = []
    for w in sorted(sums):
        first = next((m for m in CLEAR.finditer(body) if re.search(r"\b%s\b(?:\[\w+\])?\s*=" % w, m.group(1))), None)
        if not first:
            continue  # (stored by all its threads)
        rest = body[first.end():]
        # (other words cleared in the same place belong to the same group)
        while CLEAR.match(rest.lstrip()):
            rest = rest.lstrip()
            rest = rest[CLEAR.match(rest).end():]
        stop = re.search(r"\b(?:if|for|while|do)\b|&%s\b" % w, rest)
        sync = rest.find("__syncthreads()")
        if sync < 0 or (stop and stop.start() < sync):
            bad.append(w)
    return bad


FILES = sorted(os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "gr_*.hip")))


@pytest.mark.parametrize("name", FILES)
def test_cleared_sums_meet_a_barrier(name):
    with open(os.path.join(CSRC, name)) as f:
        found = list(kernels(f.read()))
    assert {k: unordered(b) for k, b in found} == {k: [] for k, _ in found}


def test_the_check_finds_a_missing_barrier():
    with open(os.path.join(CSRC, "gr_order.hip")) as f:
        body = dict(kernels(f.read()))["k_order"]
    assert {"sLow", "sArcs", "sRead"} <= set(unordered(body.replace("__syncthreads()", "", 1)))
