"""Scoring of few pairs (K and the checkpoints shared out over workgroups) against the oracle: tiles of 64 x 64 with every kind
of remainder, rows that end inside a 16-byte chunk or a pair of chunks, one part and many, and the paths that it stands next to."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _say(msg):
    print("[case] " + msg, flush=True)


def _bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def _store(rows, k, C, bits, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    out = [Q.quantize(torch.randn(rows, k, generator=g, device=DEV), bits) for _ in range(C)]
    return [o[0] for o in out], [o[2] for o in out]


def _eta(C):
    return [(-0.75) ** i for i in range(C)]


# k: 8192 (whole chunks), 8256 / 4160 / 1984 (1-/2-bit rows end inside a chunk, 4 bits inside a pair), 128 and 192 (shorter than
# a part); (1, 1) .. (129, 130): every remainder of the 64 x 64 tiles; 16 checkpoints
@pytest.mark.parametrize("bits", [8, 4, 2, 1])
@pytest.mark.parametrize("N,M,k,C", [(64, 512, 8192, 4), (1, 1, 8192, 4), (65, 70, 8256, 2), (129, 130, 4160, 3), (63, 20, 1984, 6),
                                     (40, 300, 128, 16), (7, 640, 192, 16), (100, 9, 16384, 2), (300, 33, 1024, 4)])
def test_split_codes_bit_exact(bits, N, M, k, C):
    _say("split bits=%d N=%d M=%d k=%d C=%d" % (bits, N, M, k, C))
    tc, tr = _store(N, k, C, bits, N + k)
    vc, vr = _store(M, k, C, bits, M + 1)
    got, full = Q.score(tc, tr, vc, vr, _eta(C), k, bits, want_full=True)
    host = lambda ts: [t.cpu().numpy() for t in ts]
    ref, ref_full = oracle.score(host(tc), host(tr), host(vc), host(vr), _eta(C), k, bits, want_full=True)
    np.testing.assert_array_equal(_bits(full.cpu().numpy()), _bits(ref_full))
    np.testing.assert_array_equal(_bits(got.cpu().numpy()), _bits(ref))
    assert torch.equal(Q.score(tc, tr, vc, vr, _eta(C), k, bits), got)


# a thread per column up to 1024 of them, a walk above, and by 256 threads where the rows fill the chip (8192 wavefronts, one more, and one column
# more than 256); checkpoints by four and what is left, parts by two and four, with every remainder
@pytest.mark.parametrize("bits,N,M,k,C", [(1, 3, 1023, 8192, 5), (8, 2, 1024, 4096, 7), (4, 2, 1025, 4096, 9), (2, 3, 2049, 2048, 6), (8, 70, 257, 1024, 1),
                                          (8, 70, 64, 3072, 3), (4, 5, 65, 8192, 8), (1, 819, 640, 8192, 3), (1, 820, 640, 8192, 6), (1, 1639, 257, 8192, 1),
                                          (8, 33, 70, 16384, 1), (8, 33, 70, 16384, 2), (1, 1025, 64, 8192, 1), (1, 1027, 60, 8192, 7)])
def test_split_columns_and_checkpoints(bits, N, M, k, C):
    test_split_codes_bit_exact(bits, N, M, k, C)


@pytest.mark.parametrize("N,M,k,C", [(64, 100, 8192, 4), (1, 3, 4096, 2), (130, 65, 192, 16), (33, 9, 16384, 1)])
def test_split_bfloat16(N, M, k, C):
    _say("split bfloat16 N=%d M=%d k=%d C=%d" % (N, M, k, C))
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    t16 = [Q.normalize16(torch.randn(N, k, generator=g, device=DEV)) for _ in range(C)]
    v16 = [Q.normalize16(torch.randn(M, k, generator=g, device=DEV)) for _ in range(C)]
    got, full = Q.score16(t16, v16, _eta(C), want_full=True)
    raw = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
    ref, ref_full = oracle.less16_score([raw(t) for t in t16], [raw(v) for v in v16], _eta(C), want_full=True)
    # at most k / 16 chained fp32 additions of exact products of unit rows: far inside C 2^-17
    assert np.abs(full.cpu().numpy() - ref_full).max() <= C * 2.0 ** -17
    assert np.abs(got.cpu().numpy() - ref).max() <= C * 2.0 ** -17
    assert torch.equal(Q.score16(t16, v16, _eta(C)), got)              # parts are added in a fixed order


def test_without_a_workspace_where_none_was_needed():
    """At most eight validation vectors and bit-plane codes: served without a workspace as well, with the same bits."""
    N, M, k, C, bits = 64, 8, 8192, 4, 1
    _say("no workspace, bits=1 N=64 M=8")
    tc, tr = _store(N, k, C, bits, 1)
    vc, vr = _store(M, k, C, bits, 2)
    with_ws = Q.score(tc, tr, vc, vr, _eta(C), k, bits)
    out = torch.empty(N, dtype=torch.float32, device=DEV)
    arr = lambda ts: (ctypes.c_void_p * C)(*[t.data_ptr() for t in ts])
    eta = (ctypes.c_float * C)(*_eta(C))
    rc = Q.lib().qless_score(arr(tc), arr(tr), arr(vc), arr(vr), ctypes.cast(eta, ctypes.c_void_p), C, N, M, k, bits,
                             ctypes.c_void_p(out.data_ptr()), None, None, 0, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    assert torch.equal(out, with_ws)


@pytest.mark.parametrize("bits", [1, 2, 4, 8, 16])
def test_workspace_laid_out_for_a_larger_call(bits):
    """A program lays its workspace out for the whole datastore and scores a few rows with it: the partial dot products of the few
    pairs need more (1000 x 597 here), and the call is served all the same, with the same integers in the same epilogue."""
    n, N, M, k, C = 1000, 94753, 597, 6080 if bits < 16 else 1920, 2
    _say("workspace of a larger call, bits=%d" % bits)
    arr = lambda ts: (ctypes.c_void_p * C)(*[t.data_ptr() for t in ts])
    eta = ctypes.cast((ctypes.c_float * C)(*_eta(C)), ctypes.c_void_p)
    out = torch.empty(n, dtype=torch.float32, device=DEV)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    L, ptr = Q.lib(), lambda t: ctypes.c_void_p(t.data_ptr())
    if bits == 16:
        g = torch.Generator(device=DEV)
        g.manual_seed(3)
        t16 = [Q.normalize16(torch.randn(n, k, generator=g, device=DEV)) for _ in range(C)]
        v16 = [Q.normalize16(torch.randn(M, k, generator=g, device=DEV)) for _ in range(C)]
        ws = torch.empty(L.qless_score16_workspace(N, M, k, C), dtype=torch.uint8, device=DEV)
        assert L.qless_score16(arr(t16), arr(v16), eta, C, n, M, k, ptr(out), None, ptr(ws), ws.numel(), stream) == 0
        # two sums of at most k / 16 chained fp32 additions of exact products of unit rows
        assert (out - Q.score16(t16, v16, _eta(C))).abs().max() <= C * 2.0 ** -16
        return
    tc, tr = _store(n, k, C, bits, 1)
    vc, vr = _store(M, k, C, bits, 2)
    ws = torch.empty(L.qless_score_workspace(N, M, k, bits, C) + 16, dtype=torch.uint8, device=DEV)
    assert L.qless_score(arr(tc), arr(tr), arr(vc), arr(vr), eta, C, n, M, k, bits, ptr(out), None, ptr(ws), ws.numel(), stream) == 0
    assert torch.equal(out, Q.score(tc, tr, vc, vr, _eta(C), k, bits))


# 4 bits and 81 validation vectors: streamed or tiled by k; 1 and 2 bits: streamed, popcounts (k % 128 != 0), tiled (M > 192)
@pytest.mark.parametrize("bits,M,k", [(8, 20, 4096), (8, 200, 4096), (4, 81, 8192), (4, 81, 8256), (2, 9, 8192), (2, 40, 8192),
                                      (2, 40, 1984), (1, 9, 8192), (1, 100, 8192), (1, 300, 8192), (1, 40, 1984), (16, 20, 2048),
                                      (16, 200, 2048)])
def test_norms_that_are_not_finite(bits, M, k):
    """The few pairs of a batch score what the same rows score in a large store, also where a norm is NaN or infinite."""
    n, N, C = 65, 40000, 2
    _say("norms that are not finite, bits=%d M=%d k=%d" % (bits, M, k))
    if bits == 16:
        g = torch.Generator(device=DEV)
        g.manual_seed(3)
        t16 = [Q.normalize16(torch.randn(N, k, generator=g, device=DEV)) for _ in range(C)]
        v16 = [Q.normalize16(torch.randn(M, k, generator=g, device=DEV)) for _ in range(C)]
        t16[0][7, 11] = float("nan")
        t16[1][64] = float("nan")
        few = Q.score16([t[:n].contiguous() for t in t16], v16, _eta(C))
        many = Q.score16(t16, v16, _eta(C))[:n]
        for z in range(n):
            assert bool(few[z].isnan()) == bool(many[z].isnan()) == (z in (7, 64)), z
        assert (few - many)[~many.isnan()].abs().max() <= C * 2.0 ** -16
        return
    tc, tr = _store(N, k, C, bits, 5)
    vc, vr = _store(M, k, C, bits, 6)
    tr[0][7] = float("nan")
    tr[1][64] = float("nan")
    tr[1][13] = float("inf")
    vr[0][M - 1] = float("nan")
    few = Q.score([t[:n] for t in tc], [r[:n] for r in tr], vc, vr, _eta(C), k, bits)
    many = Q.score(tc, tr, vc, vr, _eta(C), k, bits)[:n]
    np.testing.assert_array_equal(_bits(few.cpu().numpy()), _bits(many.cpu().numpy()))
