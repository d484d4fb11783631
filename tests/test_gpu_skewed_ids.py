"""Graphs whose arcs lie in a small part of the id range (numbered by degree, a
dense part beside a sparse one, trees numbered from the root): growth chunks are
cut at nodes instead of bitmap words there, so neighbouring chunks share words.
Every variant, driver and kind of job equals the oracle; and the arcs are spread,
so the numbering costs little."""
import sys
import time

import numpy as np
import pytest

import graphgen
import oracle
import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu

REF = {cd.VARIANT_FIXPOINT: oracle.decompose, cd.VARIANT_STEPS: oracle.decompose_steps,
       cd.VARIANT_CLUSTER2: oracle.decompose_cluster2}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cd.load_library()


def _edges(g):
    u = np.repeat(np.arange(g.n), np.diff(g.row_ptr.astype(np.int64)))
    keep = u < g.col
    return u[keep], g.col[keep].astype(np.int64), g.w[keep]


def _renumber(g, new):
    u, v, w = _edges(g)
    return graphgen.csr_from_edges_np(g.n, new[u], new[v], w)


def _by_degree(g):
    new = np.empty(g.n, np.int64)
    new[np.argsort(-np.diff(g.row_ptr.astype(np.int64)), kind="stable")] = np.arange(g.n)
    return _renumber(g, new)


def _tree(n, b):
    i = np.arange(1, n)
    return graphgen.csr_from_edges_np(n, (i - 1) // b, i, 1 + (i * 7919) % 1000)


def _beside(side, c, k, first):
    """A side x side mesh and a band of c nodes joined to the k nearest on either side."""
    gu, gv, gw = _edges(graphgen.grid(side, side, 10000, 3))
    bu = np.concatenate([np.arange(c - i) for i in range(1, k + 1)])
    bv = np.concatenate([np.arange(i, c) for i in range(1, k + 1)])
    bw = 1 + (bu * 31 + bv * 17) % 10000
    n = side * side
    g0, b0 = (c, 0) if first else (0, n)
    return graphgen.csr_from_edges_np(n + c, np.concatenate([gu + g0, bu + b0, [g0]]), np.concatenate([gv + g0, bv + b0, [b0]]),
                                      np.concatenate([gw, bw, [5]]))


def _star(n, at):
    i = np.delete(np.arange(n), at)
    return graphgen.csr_from_edges_np(n, np.full(n - 1, at), i, 1 + i % 777)


GRAPHS = {"rmat10": lambda: _by_degree(graphgen.rmat(10, seed=1)), "rmat13": lambda: _by_degree(graphgen.rmat(13, seed=2)),
          "tree9": lambda: _tree(5000, 9), "tree40": lambda: _tree(9001, 40), "tree700": lambda: _tree(20000, 700),
          "band_first": lambda: _beside(90, 150, 60, True), "band_last": lambda: _beside(91, 333, 50, False),
          "star_first": lambda: _star(9000, 0), "star_mid": lambda: _star(9001, 4500), "star_last": lambda: _star(9003, 9002)}
_made = {}


def _graph(name):
    if name not in _made:
        _made[name] = GRAPHS[name]()
    return _made[name]


def _skew(g):
    """Fullest of 64 equal id ranges, in average ranges."""
    rp, per = g.row_ptr.astype(np.int64), -(-g.n // 64)
    at = np.minimum(np.arange(65) * per, g.n)
    return 64 * int(np.diff(rp[at]).max()) / int(rp[-1])


KNOBS = [{}, dict(driver=cd.DRIVER_PERSISTENT), dict(pull_mode=cd.PULL_ALWAYS), dict(pull_mode=cd.PULL_NEVER), dict(grid_blocks=3),
         dict(grid_blocks=8, chunk_factor=5, local_rounds=0), dict(local_queue=64, wave_row_min=3, group_row_min=40)]


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_decompositions_equal_the_oracle(name):
    g = _graph(name)
    assert _skew(g) > 4
    dg = cd.cldiam_load_csr(g)
    for variant, ref in REF.items():
        want = ref(g, 1, 3)
        for kn in KNOBS:
            print(f"[skew] {name} n={g.n} variant={variant} {kn}", file=sys.stderr, flush=True)
            c, D, st = cd.cldiam_decompose(dg, 1, 3, variant=variant, **kn)
            assert np.array_equal(c.cpu().numpy(), want.cluster)
            assert np.array_equal(cd.u64(D), want.D)
            assert (st.stages, st.levels, st.num_clusters) == (want.stages, want.levels, want.num_clusters)
            if variant == cd.VARIANT_STEPS:
                assert (st.rounds, st.messages, st.updates) == tuple(want.work[x] for x in ("rounds", "messages", "updates"))


@pytest.mark.parametrize("driver", [cd.DRIVER_HOST, cd.DRIVER_PERSISTENT])
def test_batches_and_servers(driver):
    graphs = [_graph(n) for n in sorted(GRAPHS)] + [graphgen.grid(37, 41, 100, 1), graphgen.grid(1, 1, 1, 1)]
    dgs = [cd.cldiam_load_csr(g) for g in graphs]
    variants = [i % 3 for i in range(len(graphs))]
    want = [REF[v](g, 1, i) for i, (g, v) in enumerate(zip(graphs, variants))]
    print(f"[skew] batch of {len(graphs)}, driver {driver}", file=sys.stderr, flush=True)
    cs, Ds, _ = cd.cldiam_decompose_batch(dgs, [(1, i, 0, v, 0) for i, v in enumerate(variants)], driver)
    for c, D, w in zip(cs, Ds, want):
        assert np.array_equal(c.cpu().numpy(), w.cluster) and np.array_equal(cd.u64(D), w.D)
    if driver != cd.DRIVER_HOST:
        return
    srv = cd.Server(sum(g.n for g in graphs) // 2, 3)
    for i in reversed(range(len(graphs))):
        srv.submit(dgs[i], 1, i, i, variant=variants[i])
    found = 0
    while found < len(graphs):
        srv.step(5)
        for tag, _, _, c, D in srv.poll():
            found += 1
            assert np.array_equal(c.cpu().numpy(), want[tag].cluster) and np.array_equal(cd.u64(D), want[tag].D)
    srv.close()


def _best(g, variant):
    job, took = cd.DecomposeJob([cd.cldiam_load_csr(g)], [(1, 5, 0, variant, 0)], pull_mode=cd.PULL_NEVER), []
    for _ in range(5):
        t = time.perf_counter()
        job.run()
        took.append(time.perf_counter() - t)
    return min(took)


def test_numbering_by_degree_costs_little():
    g = graphgen.rmat(17, seed=4)
    mixed, sorted_ = _renumber(g, np.random.default_rng(1).permutation(g.n)), _by_degree(g)
    for variant in REF:
        a, b = _best(mixed, variant), _best(sorted_, variant)
        print(f"[skew] variant {variant}: {a * 1e6:.0f} us, by degree {b * 1e6:.0f}", file=sys.stderr, flush=True)
        assert b < 2.5 * a
