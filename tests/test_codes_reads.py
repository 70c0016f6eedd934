"""Host-side: the copies of the 4-bit tile kernel stay inside the train codes, and its tile shape is the one with the least padded work
on the XCD that gets the most train tiles, at the library's own prices."""
import random

import pytest

from paper_2502_01703_amd import binding as Q

SHAPES = ((256, 192), (256, 128), (512, 96))             # train rows, validation rows


@pytest.mark.parametrize("shape", range(3))
def test_copies_end_inside_the_store(shape):
    reach = Q.lib().qless_internal_codes_reach
    reach.restype, reach.argtypes = Q._i64, [Q._i64, Q._c.c_int, Q._c.c_int]
    h = SHAPES[shape][0]
    for row_bytes in (32, 64, 96, 128, 160, 192, 224, 256, 288, 320, 512):
        for tiles in (0, 1, 3):
            for rest in (1, 2, 3, 4, 5, 8, h // 2, h - 1, h):
                N = tiles * h + rest
                assert (N - 1) * row_bytes < reach(N, row_bytes, shape) <= N * row_bytes, (row_bytes, N)


def test_shape_has_the_least_work():
    shape = Q.lib().qless_internal_codes_shape
    shape.restype, shape.argtypes = Q._c.c_int, [Q._i64, Q._i32]
    pair = Q.lib().qless_internal_codes_pair
    pair.restype, pair.argtypes = Q._c.c_double, [Q._c.c_int]
    rng = random.Random(5)

    def work(N, M, i):
        (rows, cols), cost = SHAPES[i], pair(i)
        workgroups = [0] * 8
        for tile in range(-(-N // rows)):
            workgroups[tile % 8] += -(-M // cols)
        return -(-max(workgroups) // 32) * rows * cols * cost
    for N, M in [(270000, 1024), (270000, 285), (65536, 192)] + [(int(4000 * 70.0 ** rng.random()), rng.randint(65, 1024)) for _ in range(300)]:
        costs = [work(N, M, i) for i in range(3)]
        assert costs[shape(N, M)] == pytest.approx(min(costs)), (N, M)
