"""The quotient's pair table and its list where they can go wrong: cluster
counts around 16-bit ids and around what the ranking takes, more pairs than the
table holds, values that the bound skips, node counts around a bitmap word and
a workgroup's words.  Compared with the oracle's quotient of the same labels."""
import sys

import numpy as np
import pytest

import graphgen
import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


def _expected(g, cluster, D):
    """Quotient by a numpy dictionary minimum over the directed pairs."""
    centers = np.unique(cluster)
    dense = np.searchsorted(centers, cluster)
    rp = g.row_ptr.astype(np.int64)
    u = np.repeat(np.arange(g.n), np.diff(rp))
    a, b = dense[u], dense[g.col]
    val = g.w.astype(np.uint64) + D[u] + D[g.col]
    keep = a != b
    key, val = a[keep].astype(np.int64) * len(centers) + b[keep], val[keep]
    order = np.lexsort((val, key))
    key, val = key[order], val[order]
    first = np.concatenate([[True], key[1:] != key[:-1]]) if len(key) else np.zeros(0, bool)
    key, val = key[first], val[first]
    row_ptr = np.searchsorted(key, np.arange(len(centers) + 1) * len(centers))
    return centers, row_ptr, key % len(centers), val


def _labels(n, k, seed):
    """k centers, every other node with one of them; D in several ranges."""
    rng = np.random.default_rng(seed)
    centers = np.sort(rng.choice(n, size=k, replace=False))
    cluster = centers[rng.integers(0, k, n)].astype(np.int32)
    cluster[centers] = centers
    D = rng.integers(0, [10, 2**20, 2**33][seed % 3], n).astype(np.uint64)
    D[centers] = 0
    return cluster, D


GRAPHS = {"grid300": graphgen.grid(300, 271, 1000, 1), "rmat13": graphgen.rmat(13, seed=3), "rgg9000": graphgen.rgg(9000, 0, 2),
          "rmat17": graphgen.rmat(17, seed=2)}
CASES = ([("grid300", k) for k in (1, 2, 3, 64, 700, 5000, 16383, 16384, 16385, 65535, 65536, 65537, 300 * 271)]
         + [("rmat13", k) for k in (1, 2, 90, 128, 129, 5000)] + [("rgg9000", k) for k in (1, 63, 3000)]
         + [("rmat17", k) for k in (3, 150, 2000)])


@pytest.mark.parametrize("seed", [0, 1, 2])
@pytest.mark.parametrize("name,k", CASES)
def test_quotient_of_given_labels(name, k, seed):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = GRAPHS[name]
    k = min(k, g.n)
    cluster, D = _labels(g.n, k, seed)
    print(f"[quotient] {name} k={k} seed={seed}", file=sys.stderr, flush=True)
    q = cd.cldiam_build_quotient(cd.cldiam_load_csr(g), torch.from_numpy(cluster).cuda(),
                                 torch.from_numpy(D.view(np.int64)).cuda())
    centers, row_ptr, col, val = _expected(g, cluster, D)
    assert q.k == len(centers) and q.qm == len(col)
    assert np.array_equal(q.center.cpu().numpy(), centers)
    assert np.array_equal(q.row_ptr.cpu().numpy(), row_ptr)
    assert np.array_equal(q.col.cpu().numpy(), col)
    assert np.array_equal(cd.u64(q.w), val)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 4095, 4096, 4097, 8193])
def test_numbering_around_words_and_workgroups(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = graphgen.csr_from_edges_np(n, range(n - 1), range(1, n), [5] * (n - 1))
    for k in sorted({1, (n + 1) // 2, n}):
        cluster, D = _labels(n, k, 1)
        print(f"[quotient] path of {n}, k={k}", file=sys.stderr, flush=True)
        q = cd.cldiam_build_quotient(cd.cldiam_load_csr(g), torch.from_numpy(cluster).cuda(),
                                     torch.from_numpy(D.view(np.int64)).cuda())
        centers, row_ptr, col, val = _expected(g, cluster, D)
        assert np.array_equal(q.center.cpu().numpy(), centers) and np.array_equal(q.row_ptr.cpu().numpy(), row_ptr)
        assert np.array_equal(q.col.cpu().numpy(), col) and np.array_equal(cd.u64(q.w), val)
