"""Host-side: the first pass of a top-k selection stores few histograms, each of counts that fit 16 bits, where the selected keys go later."""
from paper_2502_01703_amd import binding as Q


def test_first_pass_histograms_are_few():
    parts = Q.lib().qless_internal_topk_parts
    parts.restype, parts.argtypes = Q._c.c_int, [Q._i64]
    sizes = (16385, 65535, 65536, 65537, 131071, 131072, 131073, 270000, 10 ** 6, 10 ** 7, 4 * 10 ** 8, 2 ** 32 - 1)
    for N in sizes:
        p = parts(N)
        assert 0 <= p <= 16                                  # read by every workgroup of the second pass
        assert p == 0 or N <= p * 2 * 4096 < 65536 * p       # two rounds of 4096 scores each
        assert p * 2048 <= 4096 * 8                          # the fewest padded keys
    assert parts(131072) == 16 and parts(131073) == 0
