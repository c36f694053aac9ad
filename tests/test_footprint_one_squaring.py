"""The footprint of jobs of one squaring: the fields they hold, nothing beside them."""
import ctypes

import pytest

from paper_2412_14671_amd import _lib as L


@pytest.mark.parametrize("dims", [(32, 32, 32), (160, 192, 160), (33, 9, 17)])
@pytest.mark.parametrize("N", [2, 5])
def test_one_squaring_counts_fields_alone(dims, N):
    lib = L.load()
    p = L.Params()
    lib.muster_params_default(ctypes.byref(p))
    p.K, p.iters[0] = 1, 7
    b = ctypes.c_uint64()
    assert lib.muster_footprint(N, L.DIMS(*dims), ctypes.byref(p), ctypes.byref(b)) == L.OK
    F = 3 * dims[0] * dims[1] * dims[2] * 4
    n1, P, deep = N - 1, N * (N - 1), (N - 1) * (N - 2)
    # phi, m, v; u_1 of each direction; composed pairs; pair gradients; ping-pong; coefficients
    fields = 3 * n1 + 2 * n1 + max(deep, 1) + P + 4 * n1 + P
    # the history, the job's state and the rounding of allocations
    assert b.value == fields * F + 7 * 8 + 4096 + 65536 + 16 * 256
