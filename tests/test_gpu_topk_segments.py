"""Top-k against the oracle where the ranking cuts the selected keys into segments and the compaction sums the ties before a group
itself: selected counts around 64, 256 and the segment sizes, threshold scores shared by many examples, the largest store whose ties are
not scanned and the first whose are."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [16384, 16385, 70001, 1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize("levels", [0, 40, 3])
def test_topk_segments(N, levels):
    print("[case] top-k N=%d, %s" % (N, "%d levels" % levels if levels else "distinct"), flush=True)
    s = np.random.default_rng(N + levels).standard_normal(N).astype(np.float32)
    if levels:
        s = (np.round(s * levels) / np.float32(levels)).astype(np.float32)
    dev = torch.from_numpy(s).to("cuda")
    for k_sel in (1, 63, 64, 65, 255, 257, 1000, 4095, 8193, 16384):
        idx, val = Q.topk(dev, k_sel)
        ref = oracle.topk(s, k_sel)[0]
        np.testing.assert_array_equal(idx.cpu().numpy(), ref)
        np.testing.assert_array_equal(val.cpu().numpy(), s[ref])
