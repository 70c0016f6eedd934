"""Scores by a tile kernel in a tile shape that the test names, whatever sizes the library chooses it for."""
import torch

from paper_2502_01703_amd import binding as Q

# train rows x validation rows, in the order of the kernels' tables
SHAPES = {1: ((384, 128), (512, 96), (256, 192), (256, 128)), 2: ((256, 192), (256, 128), (384, 128)), 4: ((256, 192), (256, 128), (512, 96), (192, 256)),
          8: ((192, 256), (256, 192), (256, 128), (512, 96))}
SHAPES[16] = SHAPES[8]


def score_as(tile, parts, tc, tr, vc, vr, eta, k, bits, want_full=True):
    """(score, full) of qless_score (16 bits: qless_score16; tr and vr are not read); parts: of a checkpoint's K, 1 and 2 bits only."""
    C, N, M = len(tc), tc[0].shape[0], vc[0].shape[0]
    shape = SHAPES[bits].index(tile) + (4 if bits == 2 else 0)
    size, run = Q.lib().qless_internal_score_as_workspace, Q.lib().qless_internal_score_as
    size.restype, size.argtypes = Q._sz, [Q._i64, Q._i32, Q._i32, Q._c.c_int, Q._c.c_int, Q._c.c_int]
    run.restype, run.argtypes = Q._c.c_int, [Q._c.c_int, Q._c.c_int] + Q.EXPORTS["qless_score"][1]
    ws = torch.full((size(N, M, k, bits, C, parts),), 0x5A, dtype=torch.uint8, device="cuda")
    score = torch.empty(N, device="cuda")
    full = torch.empty(N, M, device="cuda") if want_full else None
    norms = (None, None) if bits == 16 else (Q._ptr_array(tr), Q._ptr_array(vr))
    status = run(shape, parts, Q._ptr_array(tc), norms[0], Q._ptr_array(vc), norms[1], (Q._c.c_float * C)(*eta), C, N, M, k, bits,
                 score.data_ptr(), full.data_ptr() if want_full else None, ws.data_ptr(), ws.numel(), Q._stream())
    assert status == 0, status
    return score, full
