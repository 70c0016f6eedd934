"""The FP6 tile kernel of the 4-bit codes (more than 64 validation vectors) in each of its shapes, at the edges of tiles, lines and rings,
against the oracle on the rows where a tile begins or ends: integer sums, so every score bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from named_tiles import score_as
from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"
ETA = [1.0, -0.5, 0.25]


def _bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def _codes(rows, k, C, seed, extreme):
    """Any nibbles (-8 too, which no quantiser writes) or the largest ones, with norms as if they were anything."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    out = []
    for _ in range(C):
        if extreme:
            pick = torch.tensor([0x77, 0x77, 0x77, 0x88, 0x99] if extreme > 0 else [0x88, 0x88, 0x88, 0x77], dtype=torch.uint8, device=DEV)
            c = torch.empty(rows, k // 2, dtype=torch.uint8, device=DEV)
            for r in range(0, rows, 4096):
                c[r:r + 4096] = pick[torch.randint(0, len(pick), c[r:r + 4096].shape, generator=g, device=DEV)]
            c[rows // 2] = int(pick[0])
        else:
            c = torch.randint(0, 256, (rows, k // 2), generator=g, device=DEV, dtype=torch.uint8)
        out.append((c, torch.rand(rows, generator=g, device=DEV) + 0.5))
    return [o[0] for o in out], [o[1] for o in out]


def _check(N, M, k, C, extreme=0, tile=None):
    """The named tile, or what qless_score takes."""
    tc, tr = _codes(N, k, C, N + k, extreme)
    vc, vr = _codes(M, k, C, M + k + 1, extreme)
    public = Q.score(tc, tr, vc, vr, ETA[:C], k, 4)
    got, full = score_as(tile, 0, tc, tr, vc, vr, ETA[:C], k, 4) if tile else Q.score(tc, tr, vc, vr, ETA[:C], k, 4, want_full=True)
    r = {0, N // 2, N - 1}
    for h in (192, 256, 512):
        for m in (h, N // h * h):
            r.update(x for x in (m - 1, m, m + 1) if 0 <= x < N)
    r.update(range(max(0, N - 20), N))
    at = np.array(sorted(r))
    pick = torch.from_numpy(at).to(DEV)
    ref, ref_full = oracle.score([t[pick].cpu().numpy() for t in tc], [t[pick].cpu().numpy() for t in tr],
                                 [v.cpu().numpy() for v in vc], [v.cpu().numpy() for v in vr], ETA[:C], k, 4, want_full=True)
    np.testing.assert_array_equal(_bits(got[pick].cpu().numpy()), _bits(ref))
    np.testing.assert_array_equal(_bits(full[pick].cpu().numpy()), _bits(ref_full))
    assert torch.equal(full.amax(1), got)
    assert torch.equal(public, got)
    assert tile is None or torch.equal(score_as(tile, 0, tc, tr, vc, vr, ETA[:C], k, 4, want_full=False)[0], got)


# k: rows of a quarter, half and three quarters of a line, of one line, of lines and a quarter, of as many lines as the rings hold and one
# more; C: one and several; N: whole tiles, one row less, one and two more than whole tiles, fewer than a tile
@pytest.mark.parametrize("N,M,k,C,shape", [
    (33024, 192, 64, 1, (256, 192)), (33025, 191, 128, 2, (256, 192)), (65537, 380, 192, 1, (256, 192)), (49151, 192, 512, 3, (256, 192)),
    (33026, 192, 832, 2, (256, 192)), (33025, 128, 256, 1, (256, 128)), (32769, 127, 320, 3, (256, 128)), (33024, 65, 768, 2, (256, 128)),
    (32770, 128, 64, 2, (256, 128)), (131072, 96, 256, 2, (512, 96)), (130561, 95, 64, 1, (512, 96)), (131071, 96, 576, 2, (512, 96)),
    (130900, 90, 1024, 1, (512, 96)), (33024, 256, 64, 1, (192, 256)), (33025, 255, 128, 2, (192, 256)), (33023, 330, 192, 1, (192, 256)),
    (12287, 256, 512, 3, (192, 256)), (12289, 512, 832, 2, (192, 256)), (190, 256, 256, 1, (192, 256)), (193, 65, 1024, 2, (192, 256)), (200, 16500, 64, 1, None), (255, 16400, 128, 1, None)])
def test_every_shape(N, M, k, C, shape):
    print("[case] codes N=%d M=%d k=%d C=%d" % (N, M, k, C), flush=True)
    _check(N, M, k, C, tile=shape)


# the longest rows with the largest codes: sums next to 2^24 units
@pytest.mark.parametrize("extreme", [1, -1])
def test_largest_sums(extreme):
    print("[case] codes, largest sums, %d" % extreme, flush=True)
    _check(33001, 66, 65536, 1, extreme)
