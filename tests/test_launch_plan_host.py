"""The 2-D explicit plan (pf_launch_shape, no device needed) over the sizes a problem may
have: always a kernel that exists, and the rows of a wave within the grid."""
import ctypes as ct

import pytest

from paper_2601_06079_amd import _abi as A


@pytest.mark.parametrize("quad", [A.QUAD_GAUSS, A.QUAD_LOBATTO])
@pytest.mark.parametrize("bc", [A.PERIODIC, A.NOFLUX])
@pytest.mark.parametrize("model", [A.ALLEN_CAHN, A.CAHN_HILLIARD])
@pytest.mark.parametrize("dtype", [A.F32, A.F64])
def test_every_size_has_a_plan(dtype, model, bc, quad):
    L, C = A.lib(), A.host_ctx()
    for nx, ny in ((2, 2), (2, 5000), (5000, 2), (3, 7), (63, 9), (96, 96), (500, 400), (1200, 1300), (2048, 2048),
                   (9000, 9000), (2, 1 << 24), (1 << 24, 2)):
        p = A.pf_problem(2, bc, model, A.F_01, dtype, 0, (ct.c_int64 * 3)(nx, ny, 1), 1.0, 1.0, 2.0, 1.0, 0.0, 1, quad,
                         1.5)
        ks, ty, dp = ct.c_int(), ct.c_int(), ct.c_int()
        assert L.pf_launch_shape(C, ct.byref(p), ct.byref(ks), ct.byref(ty), ct.byref(dp)) == A.PF_OK
        assert 2 <= ks.value <= 4 and 1 <= ty.value <= max(ny, 48) and dp.value == 4, (nx, ny)
        again = ct.c_int(), ct.c_int()
        assert L.pf_launch_shape(C, ct.byref(p), ct.byref(again[0]), ct.byref(again[1]), ct.byref(dp)) == A.PF_OK
        assert (again[0].value, again[1].value) == (ks.value, ty.value)
