"""Host-side: the copies of the 4-bit tile kernel stay inside the train codes, and its tile shape is the one with the least padded work."""
import random

import pytest

from paper_2502_01703_amd import binding as Q

SHAPES = ((256, 192, 1.0), (256, 128, 1.19), (512, 96, 1.19))             # train rows, validation rows, cost of a pair


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
    rng = random.Random(5)

    def work(N, M, rows, cols, cost):
        workgroups = [0] * 8
        for tile in range(-(-N // rows)):
            workgroups[tile % 8] += -(-M // cols)
        return -(-max(workgroups) // 32) * rows * cols * cost
    for N, M in [(270000, 1024), (270000, 285), (65536, 192)] + [(int(4000 * 70.0 ** rng.random()), rng.randint(65, 1024)) for _ in range(300)]:
        costs = [work(N, M, *s) for s in SHAPES]
        assert costs[shape(N, M)] == pytest.approx(min(costs)), (N, M)
