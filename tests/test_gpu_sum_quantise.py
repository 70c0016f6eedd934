"""Codes of few rows straight from the projection's planes against the codes of the summed projection: the widths at which a row takes one
more thread group, numbers of planes with every remainder by eight, rows at odd offsets of P, and the last slice with two accumulators."""
import pytest
import torch

from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("k", [64, 1024, 1088, 2048, 2112, 4096, 4160, 8192, 8256, 16384, 16448])
def test_codes_of_summed_planes(k):
    print("[case] codes of summed planes k=%d" % k, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    for n, stages in ((1, 1), (1, 2), (3, 5), (2, 7), (17, 8), (33, 13), (5, 64), (1, 300)):
        d = 128 * stages
        G = torch.randn(n, d, generator=g, device=DEV).to(torch.bfloat16)
        for bits in (1, 2, 4, 8):
            P = Q.project(G, k, seed=5)
            want = Q.quantize(P, bits)
            codes, S, rn, kept = Q.project_quantize(G, k, bits, seed=5, want_P=True)
            for x, y in zip((codes, S, rn, kept), want + (P,)):
                assert torch.equal(x, y)
    if k <= 16384:                                       # (longer rows take no accumulators)
        G = torch.randn(3, 1280, generator=g, device=DEV).to(torch.bfloat16)
        other = torch.randn(3, k + 3, generator=g, device=DEV)[:, :k]
        acc = torch.empty(3, k + 1, device=DEV)[:, :k]   # rows that 16-byte loads cannot take
        for A in (acc, torch.empty(3, k, device=DEV)):
            A.copy_(torch.randn(3, k, generator=g, device=DEV))
            want = (A + Q.project(G, k, seed=7, d_offset=256)) + other
            got = Q.project_quantize_slice(G, k, 256, A, False, True, bits=8, seed=7, P_other=other)
            for x, y in zip(got, Q.quantize(want, 8)):
                assert torch.equal(x, y)
