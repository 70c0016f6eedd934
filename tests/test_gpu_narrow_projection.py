"""Projection of batches that do not fill 64-row tiles, against the oracle: row counts at the edges of the 16-, 32- and 48-row
tiles, coordinate counts at the edges of the 512- and 1024-wide ones, gradient lengths that leave the second group of wavefronts
without columns or end inside a 16-byte chunk, rows at every alignment, and the whole path's determinism."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _say(msg):
    print("[case] " + msg, flush=True)


def _gradients(n, d, pad, lead, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(n, d, generator=g) * torch.exp(torch.randn(n, 1, generator=g))
    buf = torch.zeros(n * (d + pad) + lead + 8, dtype=dtype, device=DEV)
    G = buf[lead:lead + n * (d + pad)].view(n, d + pad)[:, :d]
    G.copy_(x.to(dtype))
    return G


def _check(G, k, kind, seed):
    ref = oracle.project(G.float().cpu().to(G.dtype).contiguous(), k, kind=kind, seed=seed).astype(np.float64)
    got = Q.project(G, k, kind=kind, seed=seed)
    assert torch.equal(got, Q.project(G, k, kind=kind, seed=seed))            # fixed order of the sums
    err = np.linalg.norm(got.cpu().numpy() - ref, axis=1) / np.maximum(np.linalg.norm(ref, axis=1), 1e-300)
    # bf16: exact products, fp32 sums; fp32 input is rounded to bf16 first (2^-9 per entry, random signs)
    assert err.max() <= (1e-4 if G.dtype == torch.bfloat16 else 1e-2), err.max()
    return got


@pytest.mark.parametrize("kind", [Q.RADEMACHER, Q.GAUSSIAN])
@pytest.mark.parametrize("n,d,k", [(1, 40001, 512), (15, 33280, 576), (16, 70000, 1024), (17, 40960, 512), (32, 30080, 1088),
                                   (33, 40003, 512), (47, 25600, 1024), (48, 50000, 448), (49, 20000, 960), (96, 20480, 1024),
                                   (150, 9999, 512)])
def test_rows_and_coordinates(kind, n, d, k):
    _say("narrow projection n=%d d=%d k=%d kind=%d" % (n, d, k, kind))
    for dtype, pad, lead in ((torch.bfloat16, 0, 0), (torch.bfloat16, 3, 1), (torch.float32, 1, 0)):
        _check(_gradients(n, d, pad, lead, dtype, n + d), k, kind, 7)


@pytest.mark.parametrize("d", [1, 7, 8, 9, 127, 128, 129, 255, 256, 257, 384, 1151, 4097])
def test_short_lengths(d):
    _say("narrow projection, short rows d=%d" % d)
    for n in (1, 16, 20, 45):
        for dtype, pad, lead in ((torch.bfloat16, 0, 0), (torch.bfloat16, 1, 1), (torch.bfloat16, 8, 8), (torch.float32, 2, 1)):
            _check(_gradients(n, d, pad, lead, dtype, d), 192, Q.RADEMACHER, 3)


def test_staged_and_direct_agree():
    """The same gradients through the asynchronous copies (aligned rows) and through registers (rows at odd offsets)."""
    _say("aligned against odd row offsets, both input types, fused codes")
    for n in (5, 16, 30, 48, 64, 130):
        A = _gradients(n, 128 * 70, 0, 0, torch.bfloat16, n)
        B = _gradients(n, 128 * 70, 5, 3, torch.bfloat16, n)
        assert torch.equal(Q.project(A, 1024, seed=9), Q.project(B, 1024, seed=9))
        ca, cb = Q.project_quantize(A, 1024, 4, seed=9), Q.quantize(Q.project(B, 1024, seed=9), 4)
        for x, y in zip(ca, cb):
            assert torch.equal(x, y)
