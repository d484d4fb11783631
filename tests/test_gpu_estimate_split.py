"""The estimate's searches in their several launches: quotients around the number
of pilot searches, around those that the card holds a search for every node of,
with few and with many sources left after the pilots, in LDS and in global
memory.  Tori and rings have equal eccentricities, so no bound excludes a
source; their diameters are known in closed form, the others' from the oracle.
A ring's searches have to run side by side."""
import sys
import time

import numpy as np
import pytest

import oracle
import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cd.load_library()


def _quotient(k, u, v, w):
    """Device quotient of simple undirected edges."""
    import torch
    a, b, ww = np.concatenate([u, v]), np.concatenate([v, u]), np.concatenate([w, w]).astype(np.int64)
    order = np.lexsort((b, a))
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    rp = np.concatenate([[0], np.cumsum(np.bincount(a, minlength=k))]).astype(np.int64)
    return cd.DeviceQuotient(k, len(ww), None, t(rp), t(b[order].astype(np.int32)), t(ww[order]))


def _ring(k):
    i = np.arange(k)
    return k, i, (i + 1) % k, np.full(k, 3)


def _torus(r, c):
    at = np.arange(r * c).reshape(r, c)
    return (r * c, np.concatenate([at.ravel(), at.ravel()]),
            np.concatenate([np.roll(at, -1, 0).ravel(), np.roll(at, -1, 1).ravel()]), np.full(2 * r * c, 3))


@pytest.mark.parametrize("k", [3, 255, 256, 257, 1021, 2303, 2305, 2816, 3001])
def test_rings(k):
    print(f"[estimate] ring of {k}", file=sys.stderr, flush=True)
    assert cd.cldiam_estimate_diameter(_quotient(*_ring(k)), 1) == (3 * (k // 2), 3 * (k // 2) + 2)


@pytest.mark.parametrize("r,c", [(3, 3), (16, 16), (17, 16), (32, 40), (33, 40), (50, 60), (113, 114)])
def test_tori(r, c):
    print(f"[estimate] torus {r} x {c}", file=sys.stderr, flush=True)
    far = 3 * (r // 2 + c // 2)
    assert cd.cldiam_estimate_diameter(_quotient(*_torus(r, c)), 1) == (far, far + 2)


def _edges(k, m, seed, parts=1):
    """A random forest of `parts` trees and m edges inside them."""
    rng = np.random.default_rng(seed)
    part = np.sort(rng.integers(0, parts, k))
    first = np.searchsorted(part, part)
    i = np.arange(k)
    u, v = first + ((i - first) * rng.random(k)).astype(np.int64), i
    keep = i > first
    a, b = rng.integers(0, k, (2, m))
    same = (part[a] == part[b]) & (a != b)
    u, v = np.concatenate([u[keep], a[same]]), np.concatenate([v[keep], b[same]])
    key = np.unique(np.minimum(u, v) * k + np.maximum(u, v))
    return k, key // k, key % k, rng.integers(1, 10**6, len(key))


@pytest.mark.parametrize("k,m,parts", [(256, 300, 1), (300, 0, 40), (1000, 0, 1), (1000, 1600, 30), (2900, 0, 700), (3000, 9000, 1),
                                       (5000, 30000, 3), (7000, 4000, 900)])
def test_random_quotients(k, m, parts):
    k, u, v, w = _edges(k, m, k + m, parts)
    print(f"[estimate] random k={k} edges={len(u)} parts={parts}", file=sys.stderr, flush=True)
    phi = oracle.diameter_edges(k, u, v, w)
    assert cd.cldiam_estimate_diameter(_quotient(k, u, v, w), 2) == (phi, phi + 4)


def _best(edges):
    q = _quotient(*edges)
    job, took = cd.EstimateJob(q.k, q.qm), []
    for _ in range(6):
        t = time.perf_counter()
        job.run(q, 1)
        took.append(time.perf_counter() - t)
    return min(took)


def test_searches_run_side_by_side():
    small, large = _best(_ring(250)), _best(_ring(1000))
    print(f"[estimate] rings of 250 and 1000: {small * 1e6:.0f}, {large * 1e6:.0f} us", file=sys.stderr, flush=True)
    assert large < 6 * small    # four times the hops of a search
