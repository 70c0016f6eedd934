"""qless_score_groups: the workspace holds at most 2 GiB of the matrix (or 16 rows), and a smaller one is served with the same bits."""
import ctypes

import pytest
import torch

from paper_2502_01703_amd import binding as Q

DEV = "cuda"


@pytest.mark.parametrize("M", [1, 65, 1024, 349525, 349526, 400000, 1 << 22, (1 << 25) + 1])
def test_matrix_in_the_workspace_is_limited(M):
    for bits, k in ((1, 64), (2, 128), (4, 64), (8, 64)):
        for N in (1, 15, 1000, 270000, 1 << 24):
            matrix = max(min(N, (2 << 30) // (4 * M)), min(N, 16)) * 4 * M
            got = Q.score_groups_workspace(N, M, k, bits, 1)
            assert min(N, 16) * 4 * M <= got <= matrix + Q.score_workspace(N, M, k, bits, 1) + 512 + (256 << 20)


@pytest.mark.gpu
@pytest.mark.parametrize("bits,N,M,k", [(4, 5001, 130, 192), (8, 5001, 9, 192), (1, 5001, 300, 512), (2, 40, 200, 64), (1, 40, 400001, 64)])
def test_smaller_workspaces(bits, N, M, k):
    C, eta, T = 2, [1.0, -0.5], 3
    print("[case] score_groups in smaller workspaces, bits=%d N=%d M=%d k=%d" % (bits, N, M, k), flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    store = lambda rows: list(zip(*[Q.quantize(torch.randn(rows, k, generator=g, device=DEV), bits)[::2] for _ in range(C)]))
    (tc, tr), (vc, vr) = store(N), store(M)
    ends = [1, M // 2, M]
    full = Q.score(tc, tr, vc, vr, eta, k, bits, want_score=False, want_full=True)
    ref = Q.aggregate(full, ends, Q.AGG_MEAN)
    most, least = Q.score_groups_workspace(N, M, k, bits, C), Q.score_groups_workspace(16, M, k, bits, C)
    assert least < most
    for size in (most, (most + least) // 2, least + (most - least) // 9, least):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        got = Q.score_groups(tc, tr, vc, vr, eta, k, bits, ends, Q.AGG_MEAN, ws=ws)
        assert torch.equal(got.view(torch.int32), ref.view(torch.int32)), size
    with pytest.raises(Q.QlessError):
        Q.score_groups(tc, tr, vc, vr, eta, k, bits, ends, Q.AGG_MEAN, ws=torch.empty(16 * 4 * M, dtype=torch.uint8, device=DEV))
