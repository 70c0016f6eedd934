"""The FP4 tile kernel of the 1- and 2-bit codes (more than 64 validation vectors) in each of its shapes, with one workgroup per tile and with
the checkpoints and K shared out, at the edges of tiles, pieces and rings, against the oracle: integer sums, so every score bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from named_tiles import score_as
from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"
ETA = [1.0, -0.5, 0.25, 0.125]


def _plan(N, M, k, bits, C, share=1):
    f = Q.lib().qless_internal_fp4_plan
    f.restype, f.argtypes = None, [Q._i64, Q._i32, Q._i32, Q._c.c_int, Q._c.c_int, Q._c.c_int, Q._c.c_void_p]
    out = (Q._c.c_int * 5)()
    f(N, M, k, bits, C, share, Q._c.cast(out, Q._c.c_void_p))
    return list(out)


def _bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def _store(rows, k, C, bits, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    out = []
    for _ in range(C):
        t = torch.randn(rows, k, generator=g, device=DEV) * torch.rand(rows, 1, generator=g, device=DEV)
        t[rows // 2] = 1.0                                    # one row of equal codes: the largest sums
        out.append(Q.quantize(t, bits))
    return [o[0] for o in out], [o[2] for o in out]


def _check(N, M, k, bits, C, tile=None, parts=0, ws=None):
    """The named tile, or what qless_score takes."""
    tc, tr = _store(N, k, C, bits, N + k)
    vc, vr = _store(M, k, C, bits, M + k + 1)
    public = Q.score(tc, tr, vc, vr, ETA[:C], k, bits, ws=ws)
    if tile:
        got, full = score_as(tile, parts, tc, tr, vc, vr, ETA[:C], k, bits)
        again = score_as(tile, parts, tc, tr, vc, vr, ETA[:C], k, bits, want_full=False)[0]
    else:
        got, full = Q.score(tc, tr, vc, vr, ETA[:C], k, bits, want_full=True, ws=ws)
        again = public
    r = {0, N // 2, N - 1}
    for h in (256, 384, 512):
        for m in (h, N // h * h):
            r.update(x for x in (m - 1, m, m + 1) if 0 <= x < N)
    r.update(range(max(0, N - 20), N))
    at = np.array(sorted(r))
    pick = torch.from_numpy(at).to(DEV)
    ref, ref_full = oracle.score([t[pick].cpu().numpy() for t in tc], [t[pick].cpu().numpy() for t in tr],
                                 [v.cpu().numpy() for v in vc], [v.cpu().numpy() for v in vr], ETA[:C], k, bits, want_full=True)
    np.testing.assert_array_equal(_bits(got[pick].cpu().numpy()), _bits(ref))
    np.testing.assert_array_equal(_bits(full[pick].cpu().numpy()), _bits(ref_full))
    assert torch.equal(full.amax(1), got)
    assert torch.equal(again, got) and torch.equal(public, got)


# bits, N, M, k, C, rows and columns of the tile, parts per checkpoint (0: one workgroup walks all checkpoints), or what the call takes.  Whole tiles and pieces, rows and
# columns that end inside a tile, rows that end inside a piece, fewer rows than a tile, one piece and as many as the ring holds and more
@pytest.mark.parametrize("bits,N,M,k,C,plan", [
    (1, 22413, 488, 512, 1, (384, 128, 0)), (1, 41643, 219, 128, 2, (384, 128, 0)), (1, 39446, 193, 512, 1, (512, 96, 0)),
    (1, 36970, 218, 640, 2, None), (1, 36970, 218, 128, 1, (512, 96, 0)), (1, 22019, 284, 512, 1, (256, 192, 0)), (1, 34668, 149, 128, 1, (256, 192, 0)),
    (1, 33001, 385, 2048, 3, None), (1, 478, 198, 512, 1, (256, 128, 0)), (1, 355, 71, 128, 1, (256, 128, 0)),
    (1, 1163, 237, 1536, 3, (256, 128, 1)), (1, 2541, 100, 1152, 3, (256, 128, 1)), (1, 319, 206, 2560, 1, (256, 128, 5)),
    (1, 300, 69, 640, 3, (256, 128, 2)),
    (2, 35701, 139, 512, 1, (256, 192, 0)), (2, 32997, 129, 128, 3, None), (2, 33025, 190, 1664, 2, (256, 192, 0)), (2, 349, 65, 512, 1, (256, 128, 0)),
    (2, 301, 71, 128, 1, (256, 128, 0)), (2, 33985, 225, 512, 1, (384, 128, 0)), (2, 34208, 255, 128, 1, (384, 128, 0)),
    (2, 591, 522, 1024, 3, (256, 128, 1)), (2, 624, 495, 640, 3, (256, 128, 1)), (2, 323, 74, 1024, 2, (256, 128, 2)), (2, 305, 67, 640, 2, (256, 128, 2)),
    (2, 8192, 256, 4096, 4, (256, 128, 1))])
def test_every_shape(bits, N, M, k, C, plan):
    print("[case] fp4 bits=%d N=%d M=%d k=%d C=%d" % (bits, N, M, k, C), flush=True)
    _check(N, M, k, bits, C, *((plan[:2], plan[2]) if plan else ()))


def test_workspace_laid_out_for_a_larger_call():
    """A larger call that is not shared out needs no planes; with its workspace the smaller one is not shared out either."""
    bits, M, k, C = 2, 256, 4096, 4
    ws = torch.empty(Q.score_workspace(40000, M, k, bits, C), dtype=torch.uint8, device=DEV)
    assert ws.numel() < Q.score_workspace(8192, M, k, bits, C) and _plan(8192, M, k, bits, C)[2] == 1
    print("[case] fp4, workspace of a larger call", flush=True)
    _check(8192, M, k, bits, C, ws=ws)


def test_rows_without_finite_norms():
    """A row none of whose sums lies above -infinity scores the same whether or not its call is shared out."""
    N, M, k, bits, C = 1163, 237, 1536, 1, 3
    tc, tr = _store(N, k, C, bits, 1)
    vc, vr = _store(M, k, C, bits, 2)
    tr[0][5], tr[0][7] = float("nan"), float("inf")
    public = Q.score(tc, tr, vc, vr, ETA[:C], k, bits)
    for parts in (0, 1, 3):
        assert torch.equal(score_as((256, 128), parts, tc, tr, vc, vr, ETA[:C], k, bits)[0].view(torch.int32), public.view(torch.int32))
