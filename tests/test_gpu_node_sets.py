"""The decomposition's node sets (one bitmap word per 64 nodes) and local
queues where they can go wrong: node counts around a word and a chunk, graphs
of a batch and a server side by side, queues and grids smaller than the
frontier, rows at the tier limits.  Results have to equal the oracle's."""
import sys

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


def _path(n):
    return graphgen.csr_from_edges_np(n, range(n - 1), range(1, n), [1 + (i * 7) % 13 for i in range(n - 1)])


def _stars(hubs, leaves):
    """Hubs in a ring, each with its own leaves (rows of leaves + 2 arcs)."""
    u = [h for h in range(hubs) for _ in range(leaves)] + list(range(hubs))
    v = list(range(hubs, hubs + hubs * leaves)) + [(h + 1) % hubs for h in range(hubs)]
    w = [1 + (i * 5) % 97 for i in range(hubs * leaves)] + [400] * hubs
    e = sorted({(min(a, b), max(a, b)): c for a, b, c in zip(u, v, w) if a != b}.items())
    return graphgen.csr_from_edges_np(hubs * (leaves + 1), [k[0] for k, _ in e], [k[1] for k, _ in e],
                                      [c for _, c in e])


GRAPHS = {f"path{n}": _path(n) for n in (1, 2, 63, 64, 65, 127, 128, 129, 1023, 1025, 8193)}
GRAPHS.update(grid333x57=graphgen.grid(333, 57, 1000, 4), stars31=_stars(20, 30), stars40=_stars(20, 40),
              stars200=_stars(12, 200), rmat11=graphgen.rmat(11, seed=8))

KNOBS = [{}, dict(local_queue=64, local_rounds=64), dict(grid_blocks=3, chunk_factor=5), dict(grid_blocks=8),
         dict(local_rounds=0, bucket_width=-1.0), dict(local_cutoff=1, grid_blocks=16),
         dict(wave_row_min=2, group_row_min=30)]


def _same(got, ref):
    c, D, st = got
    assert np.array_equal(c.cpu().numpy(), ref.cluster)
    assert np.array_equal(cd.u64(D), ref.D)
    assert (st.stages, st.levels, st.delta_end, st.num_clusters, st.singletons, st.radius) == \
        (ref.stages, ref.levels, ref.delta_end, ref.num_clusters, ref.singletons, ref.radius)
    k = min(st.stages, cd.STAGE_LOG)
    assert (st.stage_uncovered, st.stage_centers, st.stage_covered) == \
        (ref.stage_uncovered[:k], ref.stage_centers[:k], ref.stage_covered[:k])


@pytest.mark.parametrize("variant", sorted(REF))
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_sets_and_queues(name, variant):
    g = GRAPHS[name]
    ref = REF[variant](g, 1, 11)
    dg = cd.cldiam_load_csr(g)
    for kn in KNOBS:
        print(f"[sets] {name} variant={variant} {kn}", file=sys.stderr, flush=True)
        _same(cd.cldiam_decompose(dg, 1, 11, variant=variant, **kn), ref)
    if variant == cd.VARIANT_FIXPOINT:
        for pull in (cd.PULL_NEVER, cd.PULL_ALWAYS):
            print(f"[sets] {name} pull={pull}", file=sys.stderr, flush=True)
            _same(cd.cldiam_decompose(dg, 1, 11, pull_mode=pull), ref)


@pytest.mark.parametrize("driver", [cd.DRIVER_HOST, cd.DRIVER_PERSISTENT])
def test_graphs_side_by_side(driver):
    """Every graph's words are its own: a batch of all of them in every variant."""
    names = sorted(GRAPHS)
    dgs = [cd.cldiam_load_csr(GRAPHS[k]) for k in names]
    variants = [(i % 3) for i in range(len(names))]
    params = [(1, 100 + i, 0, v) for i, v in enumerate(variants)]
    print(f"[sets] batch of {len(names)}, driver={driver}", file=sys.stderr, flush=True)
    cl, D, st = cd.cldiam_decompose_batch(dgs, params, driver=driver)
    for i, k in enumerate(names):
        _same((cl[i], D[i], st[i]), REF[variants[i]](GRAPHS[k], 1, 100 + i))


def test_server_holds_its_node_capacity():
    """Graphs whose node counts fill a server's capacity exactly run together."""
    sizes = [65, 129, 1, 63, 1025]
    srv = cd.Server(sum(sizes), max_graphs=len(sizes))
    print("[sets] server filled to its capacity", file=sys.stderr, flush=True)
    for i, n in enumerate(sizes):
        srv.submit(cd.cldiam_load_csr(_path(n)), 1, 7 + i, i)
    assert srv.step(1)[1] == 0   # none is left waiting
    got = {}
    for _ in range(10000):
        srv.step(4)
        for tag, st, _, c, D in srv.poll():
            got[tag] = (c, D, st)
        if len(got) == len(sizes):
            break
    srv.close()
    for i, n in enumerate(sizes):
        _same(got[i], oracle.decompose(_path(n), 1, 7 + i))
