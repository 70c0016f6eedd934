"""Host-side: the copies of the 4-bit tile kernel stay inside the train codes, and its tile shape is the one whose rounds end first
on the XCD that gets the most train tiles, at the library's own prices."""
import random

import pytest

from paper_2502_01703_amd import binding as Q

SHAPES = ((256, 192), (256, 128), (512, 96), (192, 256))             # train rows, validation rows


@pytest.mark.parametrize("shape", range(4))
def test_copies_end_inside_the_store(shape):
    reach = Q.lib().qless_internal_codes_reach
    reach.restype, reach.argtypes = Q._i64, [Q._i64, Q._c.c_int, Q._c.c_int]
    h = SHAPES[shape][0]
    for row_bytes in (32, 64, 96, 128, 160, 192, 224, 256, 288, 320, 512):
        for tiles in (0, 1, 3):
            for rest in (1, 2, 3, 4, 5, 8, h // 2, h - 1, h):
                N = tiles * h + rest
                assert (N - 1) * row_bytes < reach(N, row_bytes, shape) <= N * row_bytes, (row_bytes, N)


def _library():
    shape, price = Q.lib().qless_internal_codes_shape, Q.lib().qless_internal_codes_round
    shape.restype, shape.argtypes = Q._c.c_int, [Q._i64, Q._i32, Q._i64, Q._c.c_int]
    price.restype, price.argtypes = Q._c.c_double, [Q._c.c_int, Q._i64, Q._c.c_int]
    return shape, price


def test_shape_ends_first():
    shape, price = _library()
    rng = random.Random(5)

    def rounds(N, M, rows, cols):
        workgroups = [0] * 8
        for tile in range(-(-N // rows)):
            workgroups[tile % 8] += -(-M // cols)
        return -(-max(workgroups) // 32)
    for N, M in [(270000, 1024), (270000, 285), (65536, 192)] + [(int(4000 * 70.0 ** rng.random()), rng.randint(65, 1024)) for _ in range(300)]:
        row_bytes, C = 32 * rng.randint(1, 256), rng.randint(1, 16)
        us = [rounds(N, M, *s) * price(i, row_bytes, C) if -M % s[1] < 192 else 1e30 for i, s in enumerate(SHAPES)]
        assert us[shape(N, M, row_bytes, C)] == pytest.approx(min(us)), (N, M)


# the tile that was measured to be the fastest: one round of 192 x 256 where the others take two, 22 instead of 25, three columns of 96-wide tiles
@pytest.mark.parametrize("N,M,k,C,tile", [(11979, 985, 5952, 5, (192, 256)), (12288, 1024, 8192, 2, (192, 256)), (12000, 1000, 2048, 3, (192, 256)),
                                          (270000, 285, 8192, 4, (512, 96)), (270000, 1024, 8192, 4, (192, 256))])
def test_shape_measured_faster(N, M, k, C, tile):
    assert SHAPES[_library()[0](N, M, k // 2, C)] == tile


def test_no_shape_pads_more_than_the_workspace():
    """The workspace pads the validation rows by 191, as it did when no shape was wider than 192, so that sizes a program has kept go on to serve."""
    shape, _ = _library()
    for M in list(range(65, 1300, 7)) + [320, 321, 513, 576, 577]:
        for N in (5000, 11979, 12288, 40000, 270000):
            assert -M % SHAPES[shape(N, M, 2976, 5)][1] <= 191
