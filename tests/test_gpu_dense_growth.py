"""Growth on small graphs of long rows, where a workgroup's share is a word of
nodes or a few: complete graphs and bands around the numbers of nodes and arcs at
which that share changes, in every variant and driver, against the oracle.  All
workgroups have to take part: a growth to the fixpoint costs a few times a
growth in steps, which spreads the same rows."""
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


def _band(n, k):
    u = np.concatenate([np.arange(n - i) for i in range(1, k + 1)])
    v = np.concatenate([np.arange(i, n) for i in range(1, k + 1)])
    return graphgen.csr_from_edges_np(n, u, v, np.random.default_rng(k).integers(1, 10000, len(u)))


def _complete(n):
    u, v = np.triu_indices(n, 1)
    return graphgen.csr_from_edges_np(n, u, v, np.random.default_rng(n).integers(1, 10000, len(u)))


GRAPHS = {**{f"K{n}": (_complete, n) for n in (2, 63, 64, 65, 129, 600)},
          **{f"band{k}": (_band, 5000, k) for k in (15, 16, 17, 40, 127, 128, 129)}}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_decompositions_equal_the_oracle(name):
    g = GRAPHS[name][0](*GRAPHS[name][1:])
    dg = cd.cldiam_load_csr(g)
    for variant, ref in REF.items():
        want = ref(g, 1, 7)
        for kn in ({}, dict(driver=cd.DRIVER_PERSISTENT), dict(pull_mode=cd.PULL_ALWAYS), dict(grid_blocks=9)):
            print(f"[growth] {name} variant={variant} {kn}", file=sys.stderr, flush=True)
            c, D, st = cd.cldiam_decompose(dg, 1, 7, variant=variant, **kn)
            assert np.array_equal(c.cpu().numpy(), want.cluster)
            assert np.array_equal(cd.u64(D), want.D)
            assert (st.stages, st.levels, st.num_clusters) == (want.stages, want.levels, want.num_clusters)


def _best(dg, variant):
    job, took = cd.DecomposeJob([dg], [(1, 5, 0, variant, 0)]), []
    for _ in range(6):
        t = time.perf_counter()
        job.run()
        took.append(time.perf_counter() - t)
    return min(took)


def test_a_complete_graph_is_shared():
    dg = cd.cldiam_load_csr(_complete(3000))
    grow, steps = _best(dg, cd.VARIANT_FIXPOINT), _best(dg, cd.VARIANT_STEPS)
    print(f"[growth] K3000: {grow * 1e6:.0f} us, in steps {steps * 1e6:.0f}", file=sys.stderr, flush=True)
    assert grow < 4.2 * steps
