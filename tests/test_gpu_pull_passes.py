"""Repeated pull passes: graphs on which a level takes one pass, several, or
more than are allowed before it goes on by pushing; rows in every tier of a
scan; both drivers; graphs side by side.  Results equal the oracle's."""
import sys

import numpy as np
import pytest

import graphgen
import oracle
import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cd.load_library()


def _path(n):
    return graphgen.csr_from_edges_np(n, range(n - 1), range(1, n), [1 + (i * 7) % 13 for i in range(n - 1)])


def _hub_path(leaves):
    """A hub over the nodes of a path: the way along the path is often shorter."""
    u = [0] * leaves + list(range(1, leaves))
    v = list(range(1, leaves + 1)) + list(range(2, leaves + 1))
    w = [1 + (i * 7919) % 5000 for i in range(leaves)] + [1 + i % 3 for i in range(leaves - 1)]
    return graphgen.csr_from_edges_np(leaves + 1, u, v, w)


GRAPHS = {"path2": _path(2), "path65": _path(65), "path3000": _path(3000), "grid40x90": graphgen.grid(40, 90, 1000, 4),
          "hub33": _hub_path(33), "hub1024": _hub_path(1024), "hub1025": _hub_path(1025), "hub9000": _hub_path(9000),
          "rmat9": graphgen.rmat(9, seed=3), "rmat13": graphgen.rmat(13, seed=4)}
KNOBS = [{}, dict(wave_row_min=2, group_row_min=30), dict(grid_blocks=8, chunk_factor=3), dict(local_rounds=0)]


def _same(got, ref):
    c, D, st = got
    assert np.array_equal(c.cpu().numpy(), ref.cluster)
    assert np.array_equal(cd.u64(D), ref.D)
    assert (st.stages, st.levels, st.delta_end, st.num_clusters, st.singletons, st.radius) == \
        (ref.stages, ref.levels, ref.delta_end, ref.num_clusters, ref.singletons, ref.radius)


@pytest.mark.parametrize("delta0", [0, 1, 100000])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_passes(name, delta0):
    g = GRAPHS[name]
    ref = oracle.decompose(g, 1, 3, delta0=delta0)
    dg = cd.cldiam_load_csr(g)
    for mode in (cd.PULL_AUTO, cd.PULL_ALWAYS):
        for kn in KNOBS:
            for driver in (cd.DRIVER_HOST, cd.DRIVER_PERSISTENT):
                print(f"[pull] {name} delta0={delta0} mode={mode} {kn} driver={driver}", file=sys.stderr, flush=True)
                _same(cd.cldiam_decompose(dg, 1, 3, delta0=delta0, pull_mode=mode, driver=driver, **kn), ref)


def test_side_by_side():
    names = sorted(GRAPHS)
    dgs = [cd.cldiam_load_csr(GRAPHS[k]) for k in names]
    print(f"[pull] batch of {len(names)}", file=sys.stderr, flush=True)
    cl, D, st = cd.cldiam_decompose_batch(dgs, [(1, 50 + i, 0, 0) for i in range(len(names))], pull_mode=cd.PULL_ALWAYS)
    for i, k in enumerate(names):
        _same((cl[i], D[i], st[i]), oracle.decompose(GRAPHS[k], 1, 50 + i))
