"""Host-side: the tile shape of the wide scoring kernel is the one with the least padded work on the XCD that gets the most tiles
(consecutive train tiles go to consecutive XCDs, with all their validation tiles)."""
import random

import pytest

from paper_2502_01703_amd import binding as Q

SHAPES = ((192, 256, 1.0), (256, 192, 1.0), (256, 128, 1.06), (512, 96, 1.16))      # train rows, validation rows, cost of a pair


def _work(N, M, shape):
    rows, cols, cost = shape
    workgroups = [0] * 8
    for tile in range(-(-N // rows)):
        workgroups[tile % 8] += -(-M // cols)
    return -(-max(workgroups) // 32) * rows * cols * cost


def test_shape_has_the_least_work():
    shape = Q.lib().qless_internal_wide_shape
    shape.restype, shape.argtypes = Q._c.c_int, [Q._i64, Q._i32]
    rng = random.Random(3)
    cases = [(12384, 873), (25316, 773), (270000, 1024), (270000, 285), (65536, 512)]
    cases += [(int(4000 * 70.0 ** rng.random()), rng.randint(65, 1024)) for _ in range(300)]
    for N, M in cases:
        work = [_work(N, M, s) for s in SHAPES]
        assert work[shape(N, M)] == pytest.approx(min(work)), (N, M)
