"""Estimates of quotients with an odd number of nodes on both sides of the LDS
limit.  Past it, distances live in per-workgroup slices of global memory:
64-bit distances have to be 8-byte aligned in every slice.  A ring's diameter is known
in closed form."""
import ctypes
import sys

import numpy as np
import pytest

import paper_1506_03265_amd as cd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [3073, 3075, 12799, 12801])
def test_ring_of_an_odd_number_of_clusters(k):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    i = np.arange(k)
    col = np.sort(np.stack([(i - 1) % k, (i + 1) % k], 1), 1).reshape(-1)
    rp = torch.arange(0, 2 * k + 1, 2, dtype=torch.int64, device="cuda")
    q = cd.DeviceQuotient(k, 2 * k, None, rp, torch.from_numpy(col.astype(np.int32)).cuda(),
                          torch.full((2 * k,), 3, dtype=torch.int64, device="cuda"))
    print(f"[estimate] ring of {k}", file=sys.stderr, flush=True)
    assert cd.cldiam_estimate_diameter(q, 5) == (3 * (k // 2), 3 * (k // 2) + 10)
    phi, approx = ctypes.c_uint64(), ctypes.c_uint64()
    lib = cd.load_library()
    rc = lib.cldiam_estimate_diameter_noalloc(k, 2 * k, rp.data_ptr(), q.col.data_ptr(), q.w.data_ptr(), 5,
                                              ctypes.byref(phi), ctypes.byref(approx),
                                              torch.cuda.current_stream().cuda_stream)
    assert rc == cd.CLDIAM_OK and (phi.value, approx.value) == (3 * (k // 2), 3 * (k // 2) + 10)
