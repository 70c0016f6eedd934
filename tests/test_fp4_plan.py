"""Host-side: which kernel, tile shape and parts a call of 1- or 2-bit codes takes where the other choice was measured to be slower."""
import pytest

from paper_2502_01703_amd import binding as Q


def _plan(N, M, k, bits, C):
    f = Q.lib().qless_internal_fp4_plan
    f.restype, f.argtypes = None, [Q._i64, Q._i32, Q._i32, Q._c.c_int, Q._c.c_int, Q._c.c_int, Q._c.c_void_p]
    out = (Q._c.c_int * 5)()
    f(N, M, k, bits, C, 1, out)
    return list(out)


# us by the 128 x 64 tiles, us by the FP4 tile kernel
@pytest.mark.parametrize("bits,N,M,k,C,small,fp4", [
    (1, 843, 1024, 256, 6, 18.7, 29.8), (1, 3931, 320, 4096, 1, 20.4, 25.4), (1, 1931, 743, 256, 3, 13.5, 20.9), (1, 819, 1024, 1024, 3, 18.3, 25.5),
    (1, 10153, 384, 512, 5, 20.9, 25.9), (1, 5953, 349, 2176, 2, 24.3, 29.0), (1, 2533, 197, 1024, 3, 18.1, 21.4),
    (2, 2342, 384, 1792, 1, 16.5, 21.1), (2, 1262, 338, 2048, 1, 16.1, 18.0)])
def test_small_stores_take_the_small_tiles(bits, N, M, k, C, small, fp4):
    assert small < fp4 and not _plan(N, M, k, bits, C)[4]


@pytest.mark.parametrize("bits,N,M,k,C", [(2, 8192, 256, 16384, 4), (1, 270000, 1024, 8192, 4), (1, 270000, 285, 8192, 4), (2, 65536, 192, 8192, 4)])
def test_large_calls_take_the_fp4_tiles(bits, N, M, k, C):
    assert _plan(N, M, k, bits, C)[4]


def test_workspace_holds_planes_only_where_they_are_used():
    for bits, N, M, k, C in ((1, 843, 1024, 256, 6), (1, 10153, 384, 512, 5), (2, 2342, 384, 1792, 1)):
        assert not _plan(N, M, k, bits, C)[4]
        assert Q.score_workspace(N, M, k, bits, C) < 4 * N * M
