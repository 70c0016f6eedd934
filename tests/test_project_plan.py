"""Host-side: the projection's plan where another tile or number of d-slices was measured to be much slower."""
import ctypes

import pytest

from paper_2502_01703_amd import binding as Q


# (n, d, k, Gaussian, fp32): the tile measured as the fastest, the most d-slices that are worth their addition (us of the plan that a
# table without a price for Gaussian fp32 or for a d-slice chose, us of this one)
@pytest.mark.parametrize("n,d,k,gauss,fp32,tile,slices", [
    (48, 2621312, 2048, 1, 1, (64, 1024), 256),          # 48 x 512: 1083, 904
    (1005, 83200, 3584, 0, 1, (64, 1024), 8),            # 128 x 512: 672, 571
    (1, 169856, 320, 0, 1, (32, 512), 256),              # 16 x 512 in 443 slices: 45, 30
    (7, 116480, 512, 0, 1, (32, 512), 256),              # 16 x 512 in 455 slices: 39, 26
    (64, 1 << 27, 8192, 0, 0, (64, 1024), 32), (16, 1 << 19, 8192, 0, 0, (16, 512), 32), (128, 1 << 22, 16384, 1, 0, (128, 512), 8)])
def test_plan(n, d, k, gauss, fp32, tile, slices):
    plan = Q.lib().qless_internal_project_plan
    plan.restype, plan.argtypes = None, [Q._i64, Q._i64, Q._i32, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    out = (ctypes.c_int64 * 5)()
    plan(n, d, k, gauss, fp32, ctypes.cast(out, ctypes.c_void_p))
    assert (out[0], out[1]) == tile and out[2] <= slices, list(out)
