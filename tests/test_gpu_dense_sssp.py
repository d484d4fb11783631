"""Shortest paths on small graphs of long rows, whose frontier is a few
neighbouring nodes: distances equal the oracle's, and the arcs of a step are
spread over the card, so that nodes next to each other cost little against the
same nodes with a workgroup each."""
import sys
import time

import numpy as np
import pytest

import graphgen
import oracle
import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


def _band(n, k, seed=1):
    rng = np.random.default_rng(seed)
    u = np.concatenate([np.arange(n - i) for i in range(1, k + 1)])
    v = np.concatenate([np.arange(i, n) for i in range(1, k + 1)])
    return u, v, rng.integers(1, 10000, len(u))


def _complete(n):
    u, v = np.triu_indices(n, 1)
    return u, v, np.random.default_rng(2).integers(1, 10000, len(u))


GRAPHS = {**{f"K{n}": (n, _complete(n)) for n in (2, 31, 33, 65, 400)}, "band8": (3000, _band(3000, 8)), "band16": (3000, _band(3000, 16)),
          "band17": (3000, _band(3000, 17)), "band300": (2000, _band(2000, 300))}


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("width", [0, 700])
def test_distances_equal_the_oracle(name, width):
    _gpu()
    n, (u, v, w) = GRAPHS[name]
    g = graphgen.csr_from_edges_np(n, u, v, w)
    print(f"[sssp] {name} width {width}", file=sys.stderr, flush=True)
    dist, far = cd.cldiam_sssp_delta_stepping(cd.cldiam_load_csr(g), n // 3, width)
    ref, top = oracle.sssp(g, n // 3)
    assert np.array_equal(cd.u32(dist), ref) and far == top


def _best(g):
    import torch
    dg, took = cd.cldiam_load_csr(g), []
    for _ in range(4):
        torch.cuda.synchronize()
        t = time.perf_counter()
        cd.cldiam_sssp_delta_stepping(dg, 0)
        took.append(time.perf_counter() - t)
    return min(took)


def test_neighbouring_nodes_are_shared():
    _gpu()
    n = 2500
    u, v, w = _complete(n)
    ordered = _best(graphgen.csr_from_edges_np(n, u, v, w))
    spaced = _best(graphgen.csr_from_edges_np(64 * n, 64 * u, 64 * v, w))
    print(f"[sssp] K{n}: {ordered * 1e6:.0f} us, spaced out {spaced * 1e6:.0f}", file=sys.stderr, flush=True)
    assert ordered < 3 * spaced
