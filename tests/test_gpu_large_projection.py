"""A projection of more than 2^34 values: one thread per four of them would be 2^32 threads, more than a launch takes."""
import ctypes

import pytest
import torch

from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"


def test_more_values_than_threads_in_a_launch():
    n, k = (1 << 18) + 1, 65536
    print("[case] zero-length projection, %d x %d" % (n, k), flush=True)
    torch.cuda.empty_cache()
    P = torch.full((n, k), 3.0, dtype=torch.float32, device=DEV)             # 64 GiB
    G = torch.zeros(16, dtype=torch.bfloat16, device=DEV)
    rc = Q.lib().qless_project(ctypes.c_void_p(G.data_ptr()), Q.BF16, n, 0, 0, 0, k, Q.RADEMACHER, 1, 0, ctypes.c_void_p(P.data_ptr()), k,
                               None, 0, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    for r0 in range(0, n, 1 << 14):
        assert not P[r0:r0 + (1 << 14)].any()
    del P
    torch.cuda.empty_cache()
