"""Top-k where one workgroup selects (up to 16384 scores) and just above, on scores that cut its range of keys in every way: equal, a few values,
both zeros, denormals, infinities and NaN, one outlier; against a sort of the keys."""
import numpy as np
import pytest
import torch

from paper_2502_01703_amd import binding as Q

pytestmark = pytest.mark.gpu


def _scores(kind, N):
    r = np.random.default_rng(N + len(kind))
    s = r.standard_normal(N).astype(np.float32)
    if kind == "equal":
        s[:] = -0.25
    elif kind == "few":
        s = r.choice(np.array([-1.5, 0.0, -0.0, 2.0], np.float32), N)
    elif kind == "denormal":
        s = (s * np.float32(1e-40)).astype(np.float32)
    elif kind == "special":
        s[::3] = r.choice(np.array([np.inf, -np.inf, np.nan, -0.0, 0.0, 3e38, -3e38], np.float32), s[::3].shape)
    elif kind == "outlier":
        s = (np.float32(0.02) + s * np.float32(1e-4)).astype(np.float32)
        s[N // 2] = 0.9
    return s


def _order(s):
    u = s.view(np.uint32).copy()
    u[s == 0] = 0                                            # both zeros compare equal
    key = np.where(u & 0x80000000, ~u, u | 0x80000000).astype(np.uint32)
    return np.lexsort((np.arange(len(s)), ~key))


@pytest.mark.parametrize("kind", ["distinct", "equal", "few", "denormal", "special", "outlier"])
def test_topk_one_workgroup(kind):
    print("[case] top-k, one workgroup, %s" % kind, flush=True)
    for N in (1, 2, 63, 1024, 1025, 4095, 4096, 4097, 8192, 8193, 16383, 16384, 16385, 20001):
        s = _scores(kind, N)
        dev, order = torch.from_numpy(s).to("cuda"), _order(s)
        for k_sel in sorted({1, 2, 33, N // 20 + 1, N // 2 + 1, N - 1, N} & set(range(1, N + 1))):
            idx, val = Q.topk(dev, k_sel)
            np.testing.assert_array_equal(idx.cpu().numpy(), order[:k_sel])
            np.testing.assert_array_equal(val.cpu().numpy().view(np.uint32), s[order[:k_sel]].view(np.uint32))


@pytest.mark.parametrize("payload", [0x7FFFFFFF, 0x7FF00000, 0x7FE00001, 0x7FE00000, 0x7FDFFFFF, 0xFFFFFFFF, 0x7F800001])
def test_topk_one_workgroup_nan_payloads(payload):
    """NaN whose keys are the first or last of the 32 bits, among scores of both signs and beside the lowest key: the bin that holds the threshold
    may end past 2^32, and is cut again where fewer of them are wanted than it holds."""
    print("[case] top-k, one workgroup, NaN %08X" % payload, flush=True)
    for N in (33, 300, 2000, 4096, 8192, 16384):
        for same in (2, 10, 20):
            for lowest in (False, True):
                s = _scores("distinct", N)
                r = np.random.default_rng(N + same)
                at = r.permutation(N)
                s.view(np.uint32)[at[:same]] = payload
                if lowest:
                    s.view(np.uint32)[at[same]] = 0xFFFFFFFF
                dev, order = torch.from_numpy(s).to("cuda"), _order(s)
                for k_sel in sorted({1, same // 2, same - 1, same, same + 1, N // 2, N - 1}):
                    idx, val = Q.topk(dev, k_sel)
                    np.testing.assert_array_equal(idx.cpu().numpy(), order[:k_sel])
                    np.testing.assert_array_equal(val.cpu().numpy().view(np.uint32), s[order[:k_sel]].view(np.uint32))
