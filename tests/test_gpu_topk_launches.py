"""Top-k above 16384 scores: the first pass with a histogram per workgroup and its limits (two rounds of 4096 scores per 256 padded keys), more keys
ordered than wanted, examples with the threshold score taken by position, ranked and sorted; against a sort of the keys."""
import numpy as np
import pytest
import torch

from paper_2502_01703_amd import binding as Q
from test_gpu_topk_one import _order, _scores

pytestmark = pytest.mark.gpu


def _check(s, sels):
    dev, order = torch.from_numpy(s).to("cuda"), _order(s)
    for k_sel in sels:
        idx, val = Q.topk(dev, k_sel)
        np.testing.assert_array_equal(idx.cpu().numpy(), order[:k_sel])
        np.testing.assert_array_equal(val.cpu().numpy().view(np.uint32), s[order[:k_sel]].view(np.uint32))


@pytest.mark.parametrize("kind", ["distinct", "equal", "few", "denormal", "special", "outlier"])
def test_topk_launches(kind):
    for N in (16385, 65536, 65537, 131072, 131073, 262145):
        print("[case] top-k, launches, %s N=%d" % (kind, N), flush=True)
        # up to 256 keys more than wanted, a sixteenth of them, as many as the padding leaves (0 at 4096, 8192 and 16384); sorted above
        _check(_scores(kind, N), sorted({1, 31, 3276, 3840, 3841, 4095, 4096, 4097, 8192, 15421, 16384, 16385, N - 1, N} & set(range(1, N + 1))))


@pytest.mark.parametrize("same", [2, 256, 257, 258, 1000, 40000])
def test_topk_bucket_behind_the_last(same):
    """`same` examples share the threshold score and one of them is wanted: ordered with the others up to 256 too many, by position above."""
    N, above = 50000, 700
    print("[case] top-k, %d at the threshold" % same, flush=True)
    r = np.random.default_rng(same)
    s = r.uniform(-2, -1, N).astype(np.float32)
    at = r.permutation(N)
    s[at[:above]] = r.uniform(1, 2, above).astype(np.float32)
    s[at[above:above + same]] = 0.5
    _check(s, [above, above + 1, above + 2, above + same - 1, above + same])


def test_topk_scanned_ties():
    """More than 4096 groups of 1024 examples: the sums of the counts come from a launch of their own."""
    for kind in ("few", "equal"):
        print("[case] top-k, 4194304 + 1025, %s" % kind, flush=True)
        _check(_scores(kind, 4194304 + 1025), [1, 1000, 20000, 2000000])
