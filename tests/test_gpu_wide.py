"""The wide tile kernels of the 8-/4-bit codes and bfloat16 rows (more than 64 validation vectors) at the edges of their
tiles, stages and shapes, and the group aggregation over them, against the oracle on the rows where a tile begins or ends."""
import numpy as np
import pytest
import torch

import oracle
from named_tiles import SHAPES, score_as
from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"
ETA = [1.0, -0.5, 0.25]


def _say(msg):
    print("[case] " + msg, flush=True)


def _bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def _store(rows, k, C, bits, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    out = [Q.quantize(torch.randn(rows, k, generator=g, device=DEV), bits) for _ in range(C)]
    return [o[0] for o in out], [o[2] for o in out]


def _rows(N):
    """The first and last rows of tiles of every height, a few in between, the end of the store."""
    r = {0, N - 1}
    for h in (192, 256, 512):
        for m in (h, 7 * h, N // h * h):
            r.update(x for x in (m - 1, m, m + 1) if 0 <= x < N)
    r.update(range(max(0, N - 40), N))
    return np.array(sorted(r))


# N, M: 33001 x 129 / 513 / 97 / 257 take tiles of 192, 256, 256 and 512 rows; 49152 rows are whole tiles of each;
# k: rows of half a stage, of whole stages plus 32 and 64 bytes, of whole stages (8 bits: k bytes, 4 bits: k / 2)
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("N,M,k,C", [(33001, 129, 64, 1), (33001, 513, 192, 2), (33001, 257, 320, 2), (33001, 97, 1024, 3),
                                     (49152, 288, 512, 2), (40003, 255, 256, 1), (65537, 129, 448, 2)])
def test_wide_codes_bit_exact(bits, N, M, k, C):
    _say("wide bits=%d N=%d M=%d k=%d C=%d" % (bits, N, M, k, C))
    tc, tr = _store(N, k, C, bits, N + k)
    vc, vr = _store(M, k, C, bits, M + k)
    got, full = Q.score(tc, tr, vc, vr, ETA[:C], k, bits, want_full=True)
    at = _rows(N)
    pick = torch.from_numpy(at).to(DEV)
    ref, ref_full = oracle.score([t[pick].cpu().numpy() for t in tc], [t[pick].cpu().numpy() for t in tr],
                                 [v.cpu().numpy() for v in vc], [v.cpu().numpy() for v in vr], ETA[:C], k, bits, want_full=True)
    np.testing.assert_array_equal(_bits(got[pick].cpu().numpy()), _bits(ref))
    np.testing.assert_array_equal(_bits(full[pick].cpu().numpy()), _bits(ref_full))
    # rows that were not compared: the maximum of the matrix the kernel wrote, and the same scores without the matrix
    assert torch.equal(full.amax(1), got)
    assert torch.equal(Q.score(tc, tr, vc, vr, ETA[:C], k, bits), got)


# fewer rows than a tile, one row more than a tile, rows of half a stage and of whole stages
@pytest.mark.parametrize("N,M,k,C", [(5, 70, 64, 1), (256, 65, 128, 2), (257, 300, 192, 2), (600, 129, 64, 3), (70001, 257, 64, 1)])
def test_wide_bfloat16(N, M, k, C):
    _say("wide bfloat16 N=%d M=%d k=%d C=%d" % (N, M, k, C))
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    t16 = [Q.normalize16(torch.randn(N, k, generator=g, device=DEV)) for _ in range(C)]
    v16 = [Q.normalize16(torch.randn(M, k, generator=g, device=DEV)) for _ in range(C)]
    got, full = Q.score16(t16, v16, ETA[:C], want_full=True)
    at = _rows(N)
    pick = torch.from_numpy(at).to(DEV)
    raw = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
    ref, ref_full = oracle.less16_score([raw(t[pick]) for t in t16], [raw(v) for v in v16], ETA[:C], want_full=True)
    # fp32 sums of at most k / 16 chained additions of exact products of unit rows (|sum| <= 1): far inside C 2^-17
    assert np.abs(full[pick].cpu().numpy() - ref_full).max() <= C * 2.0 ** -17
    assert np.abs(got[pick].cpu().numpy() - ref).max() <= C * 2.0 ** -17
    assert torch.equal(full.amax(1), got)


# rows: one wavefront's 64 and its neighbours; columns: the 32-column blocks; groups shared out over wavefronts (few rows: up to one
# each, many rows: a line of columns each) or not; both kernels on either side of the line between them
@pytest.mark.parametrize("N,M,T", [(1, 1, 1), (63, 33, 5), (64, 32, 2), (64, 33, 1), (65, 64, 64), (1000, 285, 57), (2049, 290, 20),
                                   (16385, 67, 6), (16385, 66, 6), (20000, 300, 20), (20000, 256, 32), (140001, 40, 3)])
@pytest.mark.parametrize("mode", [0, 1])
def test_aggregate_edges(N, M, T, mode):
    _say("aggregate N=%d M=%d T=%d mode=%d" % (N, M, T, mode))
    g = torch.Generator(device=DEV)
    g.manual_seed(N + M)
    full = torch.randn(N, M, generator=g, device=DEV)
    full[:, M // 2] = -0.0
    cuts = sorted(np.random.default_rng(T).choice(np.arange(1, M), size=T - 1, replace=False).tolist()) + [M]
    got = Q.aggregate(full, cuts, mode).cpu().numpy()
    np.testing.assert_array_equal(_bits(got), _bits(oracle.aggregate(full.cpu().numpy(), cuts, mode)))


@pytest.mark.parametrize("bits", [4, 1])
def test_score_groups_blocks_of_rows(bits):
    """More rows than one block of the matrix in the workspace (2 GiB of fp32): the same bits as the two calls."""
    N, M, k, C = 530001, 1024, 128, 1
    _say("score_groups over two row blocks, bits=%d" % bits)
    tc, tr = _store(N, k, C, bits, 3)
    vc, vr = _store(M, k, C, bits, 4)
    ends = [1, 100, 777, 1024]
    got = Q.score_groups(tc, tr, vc, vr, ETA[:C], k, bits, ends, Q.AGG_MEAN)
    full = Q.score(tc, tr, vc, vr, ETA[:C], k, bits, want_score=False, want_full=True)
    assert torch.equal(got.view(torch.int32), Q.aggregate(full, ends, Q.AGG_MEAN).view(torch.int32))


# (N, M): the last tile holds one or two rows, in each of the four tile shapes; its rows of 32 bytes are shorter than a stage by
# three rows
@pytest.mark.parametrize("N,M", [(30145, 513), (30146, 513), (30209, 257), (30210, 257), (30209, 129), (30210, 129), (32769, 257),
                                 (32770, 257)])
def test_wide_rows_shorter_than_a_stage(N, M):
    k, bits = 64, 4
    _say("wide bits=4 k=64 N=%d M=%d" % (N, M))
    tc, tr = _store(N, k, 1, bits, N)
    vc, vr = _store(M, k, 1, bits, M)
    got, full = Q.score(tc, tr, vc, vr, ETA[:1], k, bits, want_full=True)
    at = _rows(N)
    pick = torch.from_numpy(at).to(DEV)
    ref, ref_full = oracle.score([tc[0][pick].cpu().numpy()], [tr[0][pick].cpu().numpy()], [vc[0].cpu().numpy()],
                                 [vr[0].cpu().numpy()], ETA[:1], k, bits, want_full=True)
    np.testing.assert_array_equal(_bits(got[pick].cpu().numpy()), _bits(ref))
    np.testing.assert_array_equal(_bits(full[pick].cpu().numpy()), _bits(ref_full))
    assert torch.equal(full.amax(1), got)


# whole tiles, one row less and one more, fewer rows than a tile; rows that end inside a line, of one line, of as many as the ring holds and more
@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("tile", SHAPES[8])
def test_wide_shapes(tile, bits):
    h, w = tile
    for N, M, k, C in ((8 * h, w + 1, 128, 1), (8 * h - 1, 2 * w, 192, 3), (9 * h + 1, max(w - 1, 65), 512, 2), (h + 2, w, 832, 2), (h - 1, 65, 64, 1)):
        _say("wide tile %dx%d bits=%d N=%d M=%d k=%d C=%d" % (tile + (bits, N, M, k, C)))
        if bits == 8:
            tc, tr = _store(N, k, C, 8, N + k)
            vc, vr = _store(M, k, C, 8, M + k)
            want, want_full = Q.score(tc, tr, vc, vr, ETA[:C], k, 8, want_full=True)
            got, full = score_as(tile, 0, tc, tr, vc, vr, ETA[:C], k, 8)
            assert torch.equal(got, want) and torch.equal(full, want_full)
            ref = oracle.score([t[-40:].cpu().numpy() for t in tc], [t[-40:].cpu().numpy() for t in tr], [v.cpu().numpy() for v in vc],
                               [v.cpu().numpy() for v in vr], ETA[:C], k, 8)
            np.testing.assert_array_equal(_bits(got[-40:].cpu().numpy()), _bits(ref[0] if isinstance(ref, tuple) else ref))
        else:
            g = torch.Generator(device=DEV)
            g.manual_seed(N)
            t16 = [Q.normalize16(torch.randn(N, k, generator=g, device=DEV)) for _ in range(C)]
            v16 = [Q.normalize16(torch.randn(M, k, generator=g, device=DEV)) for _ in range(C)]
            got, full = score_as(tile, 0, t16, None, v16, None, ETA[:C], k, 16)
            ref = sum(e * (t.double() @ v.double().t()) for e, t, v in zip(ETA, t16, v16))
            # fp32 sums of at most k / 16 chained additions of exact products of unit rows (|sum| <= 1): far inside C 2^-17
            assert (full.double() - ref).abs().max() <= C * 2.0 ** -17
        assert torch.equal(full.amax(1), got)
