"""The estimate's searches in global memory (quotients past the 12,800 nodes that
LDS holds): rows at every length at which their reading changes, more rows of a
workgroup's width than a pass holds, disconnected quotients, slices used again
after a larger quotient, and sizes up to the no-allocation call's limit.  The
diameters are known in closed form."""
import ctypes
import sys

import numpy as np
import pytest

import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cd.load_library()


def _grid(r, c, w=3):
    at = np.arange(r * c).reshape(r, c)
    u = np.concatenate([at[:, :-1].ravel(), at[:-1].ravel()])
    return r * c, u, np.concatenate([at[:, 1:].ravel(), at[1:].ravel()]), np.full(len(u), w), w * (r + c - 2)


def _band(k, b):
    """Unit weights; every node joined to the b nearest on either side."""
    u = np.concatenate([np.arange(k - i) for i in range(1, b + 1)])
    v = np.concatenate([np.arange(i, k) for i in range(1, b + 1)])
    return k, u, v, np.ones(len(u), np.int64), -(-(k - 1) // b)


def _hubs(leaves, hubs):
    """Every leaf joined to every hub, by its own weight."""
    a = 1 + (np.arange(leaves) * 7919) % 100003
    u, v = np.repeat(np.arange(hubs), leaves), hubs + np.tile(np.arange(leaves), hubs)
    top = np.sort(a)[-2:]
    return hubs + leaves, u, v, np.tile(a, hubs), int(top.sum())


def _parts(side, count):
    """Grids of side x side, the i-th with weights i + 1."""
    k, u, v, w, _ = _grid(side, side, 1)
    i = np.arange(count)[:, None]
    return (k * count, (u + k * i).ravel(), (v + k * i).ravel(), np.repeat(np.arange(count) + 1, len(u)),
            2 * (side - 1) * count)


def _stars(leaves, count):
    """Stars of unit weight, the last one of weight 10^12."""
    u = np.repeat(np.arange(count) * (leaves + 1), leaves)
    v = u + 1 + np.tile(np.arange(leaves), count)
    w = np.ones(len(u), np.int64)
    w[-leaves:] = 10**12
    return count * (leaves + 1), u, v, w, 2 * 10**12


CASES = {"grid120x110": lambda: _grid(120, 110), "band4": lambda: _band(12801, 4), "band20": lambda: _band(13001, 20),
         "band64": lambda: _band(14000, 64), "band65": lambda: _band(14001, 65), "hub": lambda: _hubs(12900, 1),
         "hubs": lambda: _hubs(12700, 150), "parts": lambda: _parts(12, 90), "stars": lambda: _stars(200, 70),
         "lonely": lambda: (13003, np.array([5]), np.array([13002]), np.array([11]), 11)}


def _device(k, u, v, w):
    import torch
    a, b, ww = np.concatenate([u, v]), np.concatenate([v, u]), np.concatenate([w, w]).astype(np.int64)
    order = np.lexsort((b, a))
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    rp = np.concatenate([[0], np.cumsum(np.bincount(a, minlength=k))]).astype(np.int64)
    return cd.DeviceQuotient(k, len(ww), None, t(rp), t(b[order].astype(np.int32)), t(ww[order]))


def _noalloc(q, radius):
    import torch
    phi, approx = ctypes.c_uint64(), ctypes.c_uint64()
    rc = cd.load_library().cldiam_estimate_diameter_noalloc(
        q.k, q.qm, q.row_ptr.data_ptr(), q.col.data_ptr(), q.w.data_ptr(), radius, ctypes.byref(phi),
        ctypes.byref(approx), torch.cuda.current_stream().cuda_stream)
    assert rc == cd.CLDIAM_OK
    return phi.value, approx.value


@pytest.mark.parametrize("name", sorted(CASES))
def test_known_diameters(name):
    k, u, v, w, far = CASES[name]()
    q = _device(k, u, v, w)
    print(f"[estimate] {name} k={k} arcs={q.qm}", file=sys.stderr, flush=True)
    assert cd.cldiam_estimate_diameter(q, 7) == (far, far + 14)
    assert _noalloc(q, 7) == (far, far + 14)


def test_slices_are_used_again():
    """One workspace and the static scratch, for quotients that shrink and grow."""
    job = cd.EstimateJob(32768, 1)
    for r, c in ((100, 200), (30, 30), (131, 100), (128, 256), (1, 13001), (113, 114)):
        k, u, v, w, far = _grid(r, c)
        q = _device(k, u, v, w)
        print(f"[estimate] {r} x {c}", file=sys.stderr, flush=True)
        assert job.run(q, 1) == (far, far + 2)
        assert _noalloc(q, 1) == (far, far + 2)
