"""Host-side: the copies of the 1- and 2-bit tile kernel stay inside the train codes, whatever is left for the last tile and piece."""
import pytest

from paper_2502_01703_amd import binding as Q

SHAPES = ((1, 384), (1, 512), (1, 256), (1, 256), (2, 256), (2, 256), (2, 384))


@pytest.mark.parametrize("shape", range(7))
def test_copies_end_inside_the_store(shape):
    reach = Q.lib().qless_internal_fp4_reach
    reach.restype, reach.argtypes = Q._i64, [Q._i64, Q._i32, Q._c.c_int]
    bits, h = SHAPES[shape]
    for k in (128, 256, 384, 512, 640, 1024, 1152, 1920):
        row_bytes = k * bits // 8
        for tiles in (0, 1, 3):
            for rest in (1, 2, 3, 5, 8, h // 2, h - 1, h):
                N = tiles * h + rest
                assert (N - 1) * row_bytes < reach(N, k, shape) <= N * row_bytes, (k, N)
