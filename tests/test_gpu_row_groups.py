"""Rows relaxed by groups of lanes, where the row length decides what a group
does: below, at and above a group's width and its multiples, and around the
length at which a row goes to a whole wave.  Weights make some scans stop in
the middle of a group.  Decompositions equal the oracle's, distances Dijkstra's."""
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


def _hubs(degree, hubs=30):
    """A path of hubs, each with leaves up to `degree` arcs; weights over three decades."""
    u, v, w, n = [], [], [], hubs
    for h in range(hubs):
        if h:
            u.append(h - 1); v.append(h); w.append(50 + h % 7)
        for i in range(max(0, degree - (1 if h in (0, hubs - 1) else 2))):
            u.append(h); v.append(n); w.append(1 + (i * 37 + h) % 2000)
            n += 1
    return graphgen.csr_from_edges_np(n, u, v, w)


@pytest.mark.parametrize("degree", [1, 2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 34, 64, 65, 129])
def test_row_lengths(degree):
    g = _hubs(degree)
    dg = cd.cldiam_load_csr(g)
    for variant, ref in REF.items():
        for kn in ({}, dict(local_rounds=0), dict(wave_row_min=3), dict(local_queue=64, grid_blocks=8)):
            print(f"[rows] degree={degree} variant={variant} {kn}", file=sys.stderr, flush=True)
            c, D, st = cd.cldiam_decompose(dg, 1, 5, variant=variant, **kn)
            want = ref(g, 1, 5)
            assert np.array_equal(c.cpu().numpy(), want.cluster)
            assert np.array_equal(cd.u64(D), want.D)
            assert (st.stages, st.levels, st.num_clusters) == (want.stages, want.levels, want.num_clusters)
    for width in (0, 1, 2**31):
        print(f"[rows] degree={degree} width={width}", file=sys.stderr, flush=True)
        dist, far = cd.cldiam_sssp_delta_stepping(dg, 0, width)
        want, wfar = oracle.sssp(g, 0)
        assert np.array_equal(cd.u32(dist), want)
        assert far == wfar
