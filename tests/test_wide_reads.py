"""Host-side: the copies of the wide scoring kernel stay inside the train codes, whatever is left for the last tile."""
import pytest

from paper_2502_01703_amd import binding as Q

HEIGHTS = (192, 256, 256, 512)           # train rows per tile of the four shapes


# rows of 32 bytes (4 bits, k = 64) to 512 bytes (8 bits, k = 512; bfloat16, k = 256) in steps of the shortest
@pytest.mark.parametrize("shape", range(4))
def test_copies_end_inside_the_store(shape):
    reach = Q.lib().qless_internal_wide_reach
    reach.restype, reach.argtypes = Q._i64, [Q._i64, Q._c.c_int, Q._c.c_int]
    h = HEIGHTS[shape]
    for row_bytes in (32, 64, 96, 128, 160, 192, 224, 256, 288, 320, 512):
        for tiles in (0, 1, 3):
            for rest in (1, 2, 3, 4, 5, 8, h // 2, h - 1, h):
                N = tiles * h + rest
                assert 0 < reach(N, row_bytes, shape) <= N * row_bytes, (row_bytes, N)
                # every row is read to its end
                assert reach(N, row_bytes, shape) > (N - 1) * row_bytes
