"""Host-side: the tile shape of the wide scoring kernel is the one whose rounds end first on the XCD that gets the most tiles
(consecutive train tiles go to consecutive XCDs, with all their validation tiles), and the one that was measured to be faster."""
import random

import pytest

from named_tiles import SHAPES
from paper_2502_01703_amd import binding as Q


def _library():
    shape, price = Q.lib().qless_internal_wide_shape, Q.lib().qless_internal_wide_round
    shape.restype, shape.argtypes = Q._c.c_int, [Q._i64, Q._i32, Q._i64, Q._c.c_int, Q._c.c_int]
    price.restype, price.argtypes = Q._c.c_double, [Q._c.c_int, Q._i64, Q._c.c_int, Q._c.c_int]
    return shape, price


def _rounds(N, M, tile):
    workgroups = [0] * 8
    for t in range(-(-N // tile[0])):
        workgroups[t % 8] += -(-M // tile[1])
    return -(-max(workgroups) // 32)


@pytest.mark.parametrize("bits", [8, 16])
def test_shape_ends_first(bits):
    shape, price = _library()
    rng = random.Random(3)
    cases = [(12384, 873), (25316, 773), (270000, 1024), (270000, 285), (65536, 512)]
    cases += [(int(4000 * 70.0 ** rng.random()), rng.randint(65, 1024)) for _ in range(300)]
    for N, M in cases:
        row_bytes, C = 64 * rng.randint(1, 512), rng.randint(1, 16)
        us = [_rounds(N, M, s) * price(i, row_bytes, C, bits == 16) for i, s in enumerate(SHAPES[bits])]
        assert us[shape(N, M, row_bytes, C, bits == 16)] == pytest.approx(min(us)), (N, M)


# us in the four tiles; the price of a padded pair alone chose one of more than 1.05 times the fastest's time
@pytest.mark.parametrize("bits,N,M,k,C,us", [
    (16, 65536, 512, 8192, 4, (2020, 2153, 2136, 2561)), (16, 29863, 832, 128, 3, (66.8, 59.4, 60.3, 61.2)), (16, 16935, 387, 64, 4, (27.2, 23.7, 32.5, 23.8)),
    (8, 54245, 925, 256, 4, (135.7, 125.3, 133.4, 127.5)), (8, 8494, 1024, 3712, 4, (146.3, 162.3, 220.1, 305.6)),
    (8, 26961, 612, 4096, 6, (529.4, 519.1, 568.1, 643.8))])
def test_shape_measured_faster(bits, N, M, k, C, us):
    shape, _ = _library()
    i = shape(N, M, k * bits // 8, C, bits == 16)
    assert us[i] <= 1.02 * min(us), SHAPES[bits][i]
