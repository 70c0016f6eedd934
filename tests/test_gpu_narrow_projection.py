"""Projection against the oracle in every tile shape: test_every_tile names the shape that each of its sizes takes and asks the library
for it -- full tiles and one row less, remainders of rows and coordinates, d-slices with an odd number of 128-column stages (the second
group of wavefronts is left without columns), for every input; the other tests go over row counts, coordinate counts, short
lengths and alignments whatever tile they take, and compare the copies through registers with the asynchronous ones."""
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


def _plan(n, d, k, kind, dtype):
    """Rows and columns of the tile, d-slices, stages per slice."""
    plan = Q.lib().qless_internal_project_plan
    plan.restype, plan.argtypes = None, [Q._i64, Q._i64, Q._i32, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    out = (ctypes.c_int64 * 5)()
    plan(n, d, k, int(kind == Q.GAUSSIAN), int(dtype == torch.float32), ctypes.cast(out, ctypes.c_void_p))
    return tuple(out[:4])


def _tile(n, d, k, kind, dtype):
    return _plan(n, d, k, kind, dtype)[:2]


# (tile) -> {(kind, fp32): [(n, stages of 128 columns, k), ...]}
TILES = {
    (128, 512): {(Q.RADEMACHER, 0): [(385, 3, 8256)], (Q.RADEMACHER, 1): [(128, 4097, 64)],
                 (Q.GAUSSIAN, 0): [(127, 513, 64), (128, 513, 64), (257, 193, 64), (127, 17, 8256)],
                 (Q.GAUSSIAN, 1): [(127, 513, 64), (257, 193, 64)]},
    (64, 1024): {(Q.RADEMACHER, 0): [(65, 33, 8256)], (Q.RADEMACHER, 1): [(63, 51, 8256), (257, 3, 8256)],
                 (Q.GAUSSIAN, 0): [(63, 49, 8256), (129, 13, 8256)], (Q.GAUSSIAN, 1): [(64, 49, 8256), (65, 25, 8256)]},
    (48, 1024): {(Q.RADEMACHER, 0): [(97, 37, 8256)], (Q.RADEMACHER, 1): [(48, 49, 8256), (49, 33, 8256)],
                 (Q.GAUSSIAN, 0): [(47, 49, 8256), (145, 17, 8256)]},
    (48, 512): {(Q.RADEMACHER, 0): [(48, 4097, 64), (193, 801, 64)], (Q.RADEMACHER, 1): [(47, 4097, 64)],
                (Q.GAUSSIAN, 0): [(47, 2049, 64), (48, 2049, 64), (47, 25, 8256)], (Q.GAUSSIAN, 1): [(48, 2049, 64), (145, 7, 16384)]},
    (32, 512): {(Q.RADEMACHER, 0): [(31, 513, 64), (32, 513, 64), (33, 257, 64), (31, 17, 8256)],
                (Q.RADEMACHER, 1): [(32, 513, 64), (33, 257, 64)],
                (Q.GAUSSIAN, 0): [(31, 513, 64), (32, 513, 64), (33, 257, 64), (31, 17, 8256)], (Q.GAUSSIAN, 1): [(32, 513, 64)]},
    (16, 512): {(Q.RADEMACHER, 0): [(1, 49, 8256), (15, 81, 8256), (33, 41, 8256)], (Q.RADEMACHER, 1): [(1, 49, 12352), (16, 81, 8256)],
                (Q.GAUSSIAN, 0): [(1, 49, 8256), (15, 51, 8256), (16, 51, 8256)], (Q.GAUSSIAN, 1): [(1, 81, 8256), (16, 81, 8256)]}}


@pytest.mark.parametrize("tile", sorted(TILES))
def test_every_tile(tile):
    for (kind, fp32), sizes in TILES[tile].items():
        dtype = torch.float32 if fp32 else torch.bfloat16
        for n, stages, k in sizes:
            # whole stages (bf16: asynchronous copies), the same from odd row offsets (through registers), an end inside a chunk
            for d, pad, lead in ((128 * stages, 0, 0), (128 * stages, 3, 1), (128 * stages - 5, 0, 0))[fp32:]:
                _say("projection tile %dx%d kind=%d %s n=%d d=%d k=%d pad=%d" % (tile + (kind, dtype, n, d, k, pad)))
                assert _tile(n, d, k, kind, dtype) == tile
                _check(_gradients(n, d, pad, lead, dtype, n + d), k, kind, 7)


@pytest.mark.parametrize("n,stages,per,tile", [(1000, 1, 1, (128, 512)), (1000, 2, 2, (128, 512)), (1000, 3, 3, (128, 512)),
                                               (1000, 4, 4, (128, 512)), (1000, 5, 5, (128, 512)), (640, 6, 3, (64, 1024))])
def test_gaussian_ring(n, stages, per, tile):
    """Slices of fewer, as many and more stages than the ring holds: its first fill, its last stages and the look-ups past the end."""
    _say("Gaussian ring n=%d stages=%d" % (n, stages))
    for dtype, d, pad, lead in ((torch.bfloat16, 128 * stages, 0, 0), (torch.float32, 128 * stages - 3, 1, 0)):
        assert _plan(n, d, 8256, Q.GAUSSIAN, dtype) == tile + (stages // per, per)
        _check(_gradients(n, d, pad, lead, dtype, n + d), 8256, Q.GAUSSIAN, 11)


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


@pytest.mark.parametrize("kind", [Q.RADEMACHER, Q.GAUSSIAN])
@pytest.mark.parametrize("n", [3, 17, 47, 130, 700])
def test_staged_ends(kind, n):
    """Rows staged through registers two stages ahead: slices of no, one and several whole sub-stages, with and without a rest."""
    _say("staged rows n=%d kind=%d" % (n, kind))
    for whole in (0, 1, 2, 3, 4, 5, 8):
        for rest in (0, 1, 127):
            d = 128 * whole + rest
            if d:
                _check(_gradients(n, d, 1, 1, torch.bfloat16, d), 192, kind, 13)
                _check(_gradients(n, d, 0, 0, torch.float32, d), 576, kind, 13)


@pytest.mark.parametrize("rows,fp32", [(128, 1), (128, 0), (64, 1), (64, 0)])
def test_staged_rademacher_tiles_keep_their_registers(rows, fp32):
    """Rows requested without a branch cost the 128-row tiles 8 and 30 spilled registers and up to 15 % of the time."""
    scratch = Q.lib().qless_internal_project_scratch
    scratch.restype, scratch.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int]
    _say("scratch of the %d-row tiles, fp32=%d" % (rows, fp32))
    torch.zeros(1, device=DEV)
    assert scratch(rows, fp32) == 0
