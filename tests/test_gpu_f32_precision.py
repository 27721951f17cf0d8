"""fp32 linear layers are as precise as a sum in 64 interleaved parts, at every size: on tiles, whose
contraction is summed in fp64, and on one wave per output where there is little work; at the
edges of both tile heights and of the contraction's chunks.  And fp32 attention at the number of
keys where it takes fewer waves.

Bars: a rounding is at most 2^-24 of the value.  The result of an fp64 sum is rounded once (with a
residual twice); on the other path a partial sum goes through k / 64 + 6 roundings, whose errors
are independent and of partial sums that are smaller than the total, so that for k <= 1024 the
2-norm of the error stays within two units, 1.2e-7 (one chain of k sums is off by 2e-7 at k = 256,
4e-7 at 1024).  The gated product has two such factors, of which silu passes on at most 1.1 of its
argument's relative error times a magnitude of order one, and three roundings more."""

import numpy as np
import pytest
import torch

from oracle import pkv_oracle as O
from paper_2602_02579_amd import api
from tests.test_gpu_kernels import dev, host, lcfg, rnd

pytestmark = pytest.mark.gpu

# rows, inputs, outputs: wave per output; tiles of 16 rows (also ragged ones, and contractions that
# end inside a chunk of 128 and inside a wave's part of it); tiles of 64 rows
SHAPES = [(1, 256, 512), (7, 512, 256), (3, 1024, 1024), (64, 256, 512), (151, 256, 512),
          (151, 512, 256), (17, 264, 1000), (33, 136, 2056), (220, 1000, 264), (49, 1024, 520),
          (1100, 256, 520), (1025, 136, 2056)]


def draw(device, seed, *shape, scale=1.0):
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    return torch.randn(shape, generator=gen, device=device) * scale


def off(got, want):
    return ((got.double() - want).norm() / want.norm()).item()


@pytest.mark.parametrize("m,k,n", SHAPES)
def test_linear(gpu_device, m, k, n):
    x, w, r = (draw(gpu_device, 1, m, k), draw(gpu_device, 2, n, k, scale=k ** -0.5),
               draw(gpu_device, 3, m, n))
    p = x.double() @ w.double().t()
    y = torch.full((m + 1, n), 7.0, device=gpu_device)
    api.pkv_linear_rows(x, w, None, y[:m])
    assert off(y[:m], p) <= 2.0 ** -23
    y[:m] = r
    api.pkv_linear_rows(x, w, y[:m], y[:m])
    assert off(y[:m], p + r.double()) <= 2.0 ** -23
    assert (y[m] == 7.0).all()


@pytest.mark.parametrize("m,k,n", SHAPES)
def test_gated(gpu_device, m, k, n):
    x, wg, wu = (draw(gpu_device, 1, m, k), draw(gpu_device, 2, n, k, scale=k ** -0.5),
                 draw(gpu_device, 3, n, k, scale=k ** -0.5))
    y = torch.full((m + 1, n), 7.0, device=gpu_device)
    api.pkv_swiglu_rows(x, wg, wu, y[:m])
    a, b = x.double() @ wg.double().t(), x.double() @ wu.double().t()
    assert off(y[:m], a * torch.sigmoid(a) * b) <= 2.0 ** -22
    assert (y[m] == 7.0).all()


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (8, 1, 32), (6, 2, 128)])
@pytest.mark.parametrize("n_keys", [1, 15, 17, 64, 65, 128, 129])
def test_attention_over_few_keys(gpu_device, hq, hkv, d, n_keys):
    g = np.random.default_rng(n_keys + d)
    m = min(n_keys, 21)
    cfg = lcfg("f32", hq, hkv, d)
    q, kc, vc = (rnd(s, (rows, heads, d), "f32") for s, rows, heads in
                 ((1, m, hq), (2, n_keys, hkv), (3, n_keys, hkv)))
    pos = np.sort(g.choice(n_keys, m, replace=False)).astype(np.int32)
    want, want_lse = O.sparse_row_attn(q.astype(np.float64), kc.astype(np.float64),
                                       vc.astype(np.float64), pos)
    out = torch.full((m + 1, hq, d), float("nan"), device=gpu_device)
    lse = torch.full((m + 1, hq), float("nan"), device=gpu_device)
    api.pkv_sparse_row_attn(cfg, dev(q, "f32", gpu_device), dev(kc, "f32", gpu_device),
                            dev(vc, "f32", gpu_device), torch.from_numpy(pos).to(gpu_device),
                            out[:m], lse[:m])
    # scores of a few units, d products each: a few 2^-24 sqrt(d) off, which is what a
    # probability is off by, and outputs of order one
    assert np.abs(host(out[:m]) - want).max() <= 1e-5
    assert np.abs(host(lse[:m]) - want_lse).max() <= 1e-5
    assert out[m].isnan().all() and lse[m].isnan().all()
