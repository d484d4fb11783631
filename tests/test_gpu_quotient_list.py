"""Quotients of more cluster pairs than the table holds, on graphs large enough
that every workgroup flushes several times, finds the table full and brings
pairs to the list by itself.  Compared with a numpy minimum per pair; and the
pairs come to the list together, so the call costs a few sorts of them."""
import sys
import time

import numpy as np
import pytest

import graphgen
import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cd.load_library()


def _labels(n, k, seed):
    rng = np.random.default_rng(seed)
    centers = np.sort(rng.choice(n, size=k, replace=False))
    cluster = centers[rng.integers(0, k, n)].astype(np.int32)
    cluster[centers] = centers
    D = rng.integers(0, 10**6, n).astype(np.uint64)
    D[centers] = 0
    return cluster, D


def _expected(g, cluster, D):
    centers = np.unique(cluster)
    dense = np.searchsorted(centers, cluster)
    u = np.repeat(np.arange(g.n), np.diff(g.row_ptr.astype(np.int64)))
    a, b = dense[u], dense[g.col]
    keep = a != b
    key = a[keep] * len(centers) + b[keep]
    val = (g.w.astype(np.uint64) + D[u] + D[g.col])[keep]
    order = np.lexsort((val, key))
    key, val = key[order], val[order]
    first = np.concatenate([[True], key[1:] != key[:-1]])
    key = key[first]
    return centers, np.searchsorted(key, np.arange(len(centers) + 1) * len(centers)), key % len(centers), val[first]


GRAPHS = {"grid": lambda: graphgen.grid(1100, 1000, 1000, 1), "rmat": lambda: graphgen.rmat(17, seed=5)}
_made = {}


def _graph(name):
    if name not in _made:
        _made[name] = GRAPHS[name]()
    return _made[name]


# about 8,200 pairs (just past the table), a few times as many, one per arc
@pytest.mark.parametrize("name,k", [("grid", 130), ("grid", 300), ("grid", 30000), ("rmat", 129), ("rmat", 1000), ("rmat", 70000)])
def test_pairs_past_the_table(name, k):
    import torch
    g = _graph(name)
    k = min(k, g.n)
    cluster, D = _labels(g.n, k, k)
    print(f"[quotient] {name} k={k}", file=sys.stderr, flush=True)
    q = cd.cldiam_build_quotient(cd.cldiam_load_csr(g), torch.from_numpy(cluster).cuda(),
                                 torch.from_numpy(D.view(np.int64)).cuda())
    centers, row_ptr, col, val = _expected(g, cluster, D)
    assert q.k == k and q.qm == len(col)
    assert np.array_equal(q.center.cpu().numpy(), centers) and np.array_equal(q.row_ptr.cpu().numpy(), row_ptr)
    assert np.array_equal(q.col.cpu().numpy(), col) and np.array_equal(cd.u64(q.w), val)


def _best(fn):
    import torch
    took = []
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        took.append(time.perf_counter() - t)
    return min(took[1:])


def test_listed_pairs_cost_a_few_sorts():
    import torch
    g = _graph("grid")
    cluster, D = _labels(g.n, 30000, 1)
    job = cd.QuotientJob(cd.cldiam_load_csr(g))
    cluster, D = torch.from_numpy(cluster).cuda(), torch.from_numpy(D.view(np.int64)).cuda()
    pairs = torch.randint(0, 2**30, (g.m,), device="cuda")
    sort, quotient = _best(lambda: torch.sort(pairs)), _best(lambda: job.run(cluster, D))
    print(f"[quotient] {g.m} pairs: {quotient * 1e6:.0f} us, sorted in {sort * 1e6:.0f}", file=sys.stderr, flush=True)
    assert quotient < 12 * sort
