"""The one-workgroup top-k on vectors many of whose scores share a value, everywhere or only in a
part of the vector, and with thresholds in, just above and just below such a value: the indices
against the oracle bit by bit.  And NaNs: k different indices, in the order of their
bits."""

import numpy as np
import pytest
import torch

from oracle import pkv_oracle as O
from paper_2602_02579_amd import api
from tests.test_gpu_kernels import run_topk

pytestmark = pytest.mark.gpu

# both sides of the length from which shared keys are looked for, and of the instantiations
LENGTHS = [64, 2048, 2049, 8192, 8193, 20001, 32768, 65533]


def vector(kind, n, g):
    s = g.standard_normal(n).astype(np.float32)
    if kind == "zeros":           # scores that underflowed, one in fifty did not
        return np.where(g.random(n) < 0.02, np.exp(s), 0.0).astype(np.float32)
    if kind == "three":
        return g.choice(np.float32([-1.0, 0.25, 2.0]), n, p=[0.45, 0.4, 0.15])
    if kind == "tail":            # an ordinary first half, and one value behind it
        s[n // 2:] = 0.5
        return s
    if kind == "signs":           # -0.0 and +0.0 are one value
        return np.where(g.random(n) < 0.5, np.float32(0.0), np.float32(-0.0)) * np.abs(s).round()
    return np.floor(4 * s).astype(np.float32)      # "few": some 25 values


@pytest.mark.parametrize("kind", ["zeros", "three", "tail", "signs", "few"])
@pytest.mark.parametrize("n", LENGTHS)
def test_ties(gpu_device, kind, n):
    s = vector(kind, n, np.random.default_rng(n))
    most = int(np.unique(s, return_counts=True)[1].max())
    above = int(np.count_nonzero(s > 0.5))
    ks = {1, n // 5, above, above + 1, most, n - 1, n}
    for k in sorted(k for k in ks if 1 <= k <= n):
        assert np.array_equal(run_topk(s, k, gpu_device), O.topk_select(s, k)), k


@pytest.mark.parametrize("bits", [0x7fc00000, 0xffc00000, 0x7fffffff, 0xffffffff])
@pytest.mark.parametrize("n", [100, 5000, 32767])
def test_nan_scores_give_indices_of_the_vector(gpu_device, bits, n):
    s = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    s[::3] = np.uint32(bits).view(np.float32)
    score = torch.from_numpy(s).to(gpu_device)
    for k in (1, n // 3, n - 1, n):
        idx = torch.full((k + 4,), -7, dtype=torch.int32, device=gpu_device)
        api.pkv_topk_select(score, k, idx)
        got = idx.cpu().numpy()
        assert (got[k:] == -7).all()
        assert got[0] >= 0 and got[k - 1] < n and (np.diff(got[:k]) > 0).all()


@pytest.mark.parametrize("n", [100, 5000, 32767])
def test_nan_payloads_order_as_in_the_kernel_for_any_vector(gpu_device, n):
    """NaNs of different bits are different keys, also at both ends of their range.  An address
    that is no multiple of 16 takes the kernel for any vector."""
    g = np.random.default_rng(n)
    s = g.standard_normal(n).astype(np.float32)
    bits = np.uint32([0x7fc00000, 0x7fdfffff, 0x7fe00000, 0x7ffffffe, 0x7fffffff,
                      0xffc00000, 0xfffffffe, 0xffffffff])
    at = g.random(n) < 0.6
    s[at] = g.choice(bits, int(at.sum())).view(np.float32)
    plain = torch.from_numpy(s).to(gpu_device)
    moved = torch.empty(n + 1, dtype=torch.float32, device=gpu_device)[1:].copy_(plain)
    assert plain.data_ptr() % 16 == 0 and moved.data_ptr() % 16 != 0
    u = s.view(np.uint32).astype(np.int64)
    keys = np.where(u & 0x80000000, u ^ 0xffffffff, u | 0x80000000)
    for k in sorted({1, n // 20, n // 10, n // 5, n // 3, n // 2, (3 * n) // 4, n - 2, n}):
        got = []
        for score in (plain, moved):
            idx = torch.empty(k, dtype=torch.int32, device=gpu_device)
            api.pkv_topk_select(score, k, idx)
            got.append(idx.cpu().numpy())
        want = np.sort(np.lexsort((np.arange(n), -keys))[:k])
        assert np.array_equal(got[0], want) and np.array_equal(got[1], want), k
