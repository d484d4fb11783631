"""Ingest at the sizes where it can go wrong: row lengths around every sorting
class, rows and runs of empty rows across validation tiles, and each way in
which a CSR can be asymmetric, whichever of an edge's two rows is the longer.
Packed rows have to equal a host sort; a malformed CSR has to be refused."""
import sys

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


def _hubs(degrees, pad):
    """A hub of each degree, its leaves its own, and `pad` nodes without arcs
    after every hub's leaves; weights repeat so that columns decide."""
    u, v, w, n = [], [], [], 0
    for i, d in enumerate(degrees):
        u += [n] * d
        v += range(n + 1, n + 1 + d)
        w += [1 + (j * 2654435761 + i) % 1009 for j in range(d)]
        n += 1 + d + pad
    return graphgen.csr_from_edges_np(max(n, 1), u, v, w)


def _expected(g):
    rp = g.row_ptr.astype(np.int64)
    row = np.repeat(np.arange(g.n), np.diff(rp))
    arcs = (g.w.astype(np.uint64) << np.uint64(32)) | g.col.astype(np.uint64)
    return arcs[np.lexsort((arcs, row))]


CASES = {"classes": _hubs([1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 66, 127, 128, 129, 255, 256, 257, 1023, 2047, 2048, 2049,
                           4097, 8191, 8192, 8193, 20000], 3),
         "tiles": _hubs([2047, 1, 2048, 2049, 2], 0), "gaps": _hubs([5, 700, 3000], 5000), "one": _hubs([], 0),
         "rmat12": graphgen.rmat(12, seed=9), "grid": graphgen.grid(97, 61, 50, 2)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_rows_are_sorted(name):
    g = CASES[name]
    print(f"[ingest] {name} n={g.n} m={g.m}", file=sys.stderr, flush=True)
    dg = cd.cldiam_load_csr(g)
    assert np.array_equal(cd.u64(dg.arcs)[:g.m], _expected(g))
    assert dg.weight_sum == int(g.w.astype(np.int64).sum())


def _without(g, at):
    """g without arc `at` (its reverse stays)."""
    rp = g.row_ptr.astype(np.int64).copy()
    row = int(np.searchsorted(rp, at, side="right") - 1)
    rp[row + 1:] -= 1
    return graphgen.Graph(g.n, rp, np.delete(g.col, at), np.delete(g.w, at))


@pytest.mark.parametrize("side", ["hub", "leaf"])
@pytest.mark.parametrize("what", ["missing", "weight", "column"])
def test_asymmetry_is_found_on_either_side(what, side):
    g = _hubs([40, 3000, 5], 2)
    rp = g.row_ptr.astype(np.int64)
    hub = 43                                   # the second hub, 3000 arcs
    assert rp[hub + 1] - rp[hub] == 3000
    at = int(rp[hub]) + 1234 if side == "hub" else int(rp[hub + 1 + 1234])
    print(f"[ingest] {what} on the {side}'s side", file=sys.stderr, flush=True)
    if what == "missing":
        bad = _without(g, at)
    else:
        bad = graphgen.Graph(g.n, g.row_ptr.copy(), g.col.copy(), g.w.copy())
        if what == "weight":
            bad.w[at] += 1
        elif side == "hub":
            bad.col[int(rp[hub + 1]) - 1] = g.n - 1    # the hub's last leaf becomes a node without arcs
        else:
            bad.col[at] = hub + 1                       # the leaf names its neighbour instead of the hub
    with pytest.raises(cd.CldiamError) as e:
        cd.cldiam_load_csr(bad)
    assert e.value.status == cd.CLDIAM_EINVAL and "malformed CSR" in str(e.value)


def test_malformed_offsets_are_refused():
    g = CASES["rmat12"]
    for where, by in ((5, -10**6), (g.n // 2, 10**7), (g.n, 1), (0, 1)):
        rp = g.row_ptr.astype(np.int64).copy()
        rp[where] += by
        print(f"[ingest] offset {where} off by {by}", file=sys.stderr, flush=True)
        with pytest.raises(cd.CldiamError) as e:
            cd.cldiam_load_csr(graphgen.Graph(g.n, rp, g.col, g.w))
        assert e.value.status == cd.CLDIAM_EINVAL and "row offsets" in str(e.value)
