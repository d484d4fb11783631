"""Ingest of graphs with long runs of nodes without arcs (ids taken over from a
larger graph): before, amid and after the arcs, up to and past the number of
rows that a validation tile visits one by one.  Packed rows have to equal a
host sort, and such a run must not be left to one workgroup: the ingest takes
about as long as with the same nodes and arcs spread evenly."""
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


def _spaced(g, new, n):
    """g's edges between the nodes new[0] < new[1] < ... of n."""
    rp = g.row_ptr.astype(np.int64)
    deg = np.zeros(n, np.int64)
    deg[new] = np.diff(rp)
    return graphgen.Graph(n, np.concatenate([[0], np.cumsum(deg)]), new[g.col].astype(np.int32), g.w.copy())


def _run(g, at, gap):
    """g with a run of `gap` nodes without arcs after its first `at` nodes."""
    i = np.arange(g.n)
    return _spaced(g, np.where(i < at, i, i + gap), g.n + gap)


GRID = graphgen.grid(53, 47, 1000, 3)
CASES = {**{f"amid{gap}": _run(GRID, 1200, gap) for gap in (13000, 16383, 16384, 16385, 20000, 300000)},
         "before": _run(GRID, 0, 200000), "after": _run(GRID, GRID.n, 200000),
         "two": _run(_run(GRID, 700, 40000), 41000, 50000), "every": _spaced(GRID, 100 * np.arange(GRID.n) + 7, 100 * GRID.n + 9)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_rows_are_sorted_across_runs_of_empty_rows(name):
    g = CASES[name]
    print(f"[ingest] {name} n={g.n} m={g.m}", file=sys.stderr, flush=True)
    dg = cd.cldiam_load_csr(g)
    row = np.repeat(np.arange(g.n), np.diff(g.row_ptr.astype(np.int64)))
    arcs = (g.w.astype(np.uint64) << np.uint64(32)) | g.col.astype(np.uint64)
    assert np.array_equal(cd.u64(dg.arcs)[:g.m], arcs[np.lexsort((arcs, row))])
    assert dg.weight_sum == int(g.w.astype(np.int64).sum())


def _best(g):
    """Least time of five ingests of a device-resident CSR."""
    import torch
    rp, col, w = cd.to_device(g)
    took = []
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        cd.cldiam_load_csr_device(g.n, g.m, rp, col, w)
        took.append(time.perf_counter() - t)
    return min(took[1:])


@pytest.mark.parametrize("where", ["amid", "after"])
def test_a_run_of_empty_rows_is_shared(where):
    base, more = graphgen.grid(300, 300, 1000, 1), 1 << 24
    every = more // base.n + 1
    spread = _best(_spaced(base, every * np.arange(base.n), every * base.n))
    run = _best(_run(base, base.n // 2 if where == "amid" else base.n, (every - 1) * base.n))
    print(f"[ingest] {where}: {run * 1e6:.0f} us, spread {spread * 1e6:.0f} us", file=sys.stderr, flush=True)
    assert run < 5 * spread
