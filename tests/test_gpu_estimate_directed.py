"""Estimates of quotients that are not symmetric: the largest finite distance of
an ordered pair.  A node that others reach quickly may itself be far from them,
which a bound on its eccentricity taken from theirs would hide."""
import sys

import numpy as np
import pytest
from scipy.sparse import csr_matrix
from scipy.sparse.csgraph import shortest_path

import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


def _arcs(k, arcs):
    """Row offsets, columns and weights of a dict {(u, v): w}."""
    key = np.array(sorted(arcs), dtype=np.int64).reshape(-1, 2)
    w = np.array([arcs[tuple(x)] for x in key.tolist()], dtype=np.int64)
    rp = np.zeros(k + 1, np.int64)
    np.add.at(rp, key[:, 0] + 1, 1)
    return np.cumsum(rp), key[:, 1].astype(np.int32), w


def _core(k, far):
    """A tree both ways, and from node `far` one long arc only."""
    arcs = {}
    for i in range(1, k):
        p = (i - 1) // 8
        arcs[(p, i)] = arcs[(i, p)] = 1 + i % 5
    for (u, v) in list(arcs):
        if u == far:
            arcs[(u, v)] = 10**6
    return arcs


def _cases():
    yield "ring", 601, {(i, (i + 1) % 601): 1 + i % 7 for i in range(601)}
    yield "way_down", 500, {(i, i + 1): 3 for i in range(499)}
    for far in (699, 650, 601, 555, 502, 443, 399, 333):   # leaves of the tree
        yield f"far{far}", 700, _core(700, far)
    yield "unsorted", 700, _core(700, 620)


@pytest.mark.parametrize("name,k,arcs", list(_cases()), ids=lambda x: x if isinstance(x, str) else "")
def test_largest_distance_of_an_ordered_pair(name, k, arcs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rp, col, w = _arcs(k, arcs)
    d = shortest_path(csr_matrix((w.astype(float), col, rp), shape=(k, k)))
    far = int(d[np.isfinite(d)].max())
    if name == "unsorted":
        for u in range(k):
            col[rp[u]:rp[u + 1]] = col[rp[u]:rp[u + 1]][::-1]
            w[rp[u]:rp[u + 1]] = w[rp[u]:rp[u + 1]][::-1]
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    print(f"[estimate] {name} k={k} arcs={len(col)}", file=sys.stderr, flush=True)
    q = cd.DeviceQuotient(k, len(col), None, t(rp), t(col), t(w))
    assert cd.cldiam_estimate_diameter(q, 2) == (far, far + 4)
