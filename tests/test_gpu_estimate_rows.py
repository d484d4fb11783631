"""The all-pairs step at the sizes where it can go wrong: rows at the edges of
a lane group and of the whole-workgroup form, more wide rows than a pass holds,
node counts around a bitmap word, quotients around the size that LDS holds
whole, disconnected ones.
Compared with the oracle's exact diameter."""
import sys

import numpy as np
import pytest

import oracle
import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


def _quotient(k, edges):
    """Device quotient of an undirected edge dict {(a, b): w}, a < b."""
    import torch
    a = np.array([e[0] for e in edges], dtype=np.int64)
    b = np.array([e[1] for e in edges], dtype=np.int64)
    w = np.array(list(edges.values()), dtype=np.int64)
    src, dst, ww = np.concatenate([a, b]), np.concatenate([b, a]), np.concatenate([w, w])
    order = np.lexsort((dst, src))
    rp = np.zeros(k + 1, dtype=np.int64)
    np.add.at(rp, src + 1, 1)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return (cd.DeviceQuotient(k, len(ww), None, t(np.cumsum(rp)), t(dst[order].astype(np.int32)), t(ww[order])), a, b, w)


def _star(leaves, hubs):
    """`hubs` hubs in a ring, each joined to the same leaves: hub rows of leaves + 2 arcs."""
    e = {}
    for h in range(hubs):
        for i in range(leaves):
            e[(h, hubs + i)] = 1 + (i * 7919 + h * 31) % 1000
    for h in range(hubs):
        if h + 1 < hubs:
            e[(h, h + 1)] = 2**33 + h
    return hubs + leaves, e


def _random(k, m, seed):
    rng = np.random.default_rng(seed)
    e = {((i - 1) // 2, i): int(rng.integers(1, 2**34)) for i in range(1, k)}   # a binary tree and m more
    for _ in range(m):
        a, b = sorted(rng.integers(0, k, 2).tolist())
        if a != b:
            e.setdefault((a, b), int(rng.integers(1, 2**34)))
    return k, e


def _parts(k):
    return k, {(i, i + 1): i + 1 for i in range(k - 1) if i % 5 != 4}


CASES = {"one": (1, {}), "pair": (2, {(0, 1): 9}), "lonely": (33, {}), "parts": _parts(64),
         **{f"rand{k}": _random(k, 3 * k, k) for k in (31, 32, 33, 65, 257, 1000)},
         **{f"star{n}": _star(n, 1) for n in (7, 8, 9, 127, 128, 129, 700)}, "hubs": _star(140, 150),
         "resident_limit": _random(2240, 4700, 5), "dense": _random(300, 40000, 6), "past_resident": _random(3073, 6000, 5)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_estimate_equals_the_oracle(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    k, edges = CASES[name]
    q, a, b, w = _quotient(k, edges)
    print(f"[estimate] {name} k={k} arcs={q.qm}", file=sys.stderr, flush=True)
    phi = oracle.diameter_edges(k, a, b, w)
    assert cd.cldiam_estimate_diameter(q, 3) == (phi, phi + 6)
