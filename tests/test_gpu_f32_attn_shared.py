"""fp32 attention whose tiles of 16 columns are shared by four, two or one workgroup, each with its
elements of the head: at and beyond the counts of tiles where that changes, for every head
dimension of the kernel, with a cache and with chunks that attend within themselves."""

import numpy as np
import pytest
import torch

from oracle import pkv_oracle as O
from paper_2602_02579_amd import api
from tests.test_gpu_f32_tiles import BAR
from tests.test_gpu_kernels import dev, host, lcfg, rel_err, rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n_keys,hq,hkv,d,chunk", [
    (33, 140, 4, 4, 64, 0),                                   # four
    (256, 300, 4, 4, 64, 0), (257, 300, 4, 4, 64, 0),         # 64 and 68 tiles: four, two
    (512, 530, 4, 4, 64, 0), (513, 530, 4, 4, 64, 0),         # 128 and 132: two, one
    (7, 65, 8, 2, 128, 0), (600, 620, 2, 2, 128, 0),          # four, two
    (40, 200, 4, 2, 32, 0),                                   # two at most
    (140, 140, 4, 4, 64, 139), (300, 300, 4, 4, 64, 150)])    # chunks, the last of one row
def test_shared_tiles(gpu_device, m, n_keys, hq, hkv, d, chunk):
    cfg = lcfg("f32", hq, hkv, d)
    q, k, v = rnd(1, (m, hq, d), "f32"), rnd(2, (n_keys, hkv, d), "f32"), rnd(3, (n_keys, hkv, d), "f32")
    dq, dk, dv = (dev(t, "f32", gpu_device) for t in (q, k, v))
    if chunk:
        pos = np.arange(m, dtype=np.int32) % chunk
    else:
        pos = np.sort(np.random.default_rng(m).integers(0, n_keys, m)).astype(np.int32)
        pos[-1] = n_keys - 1
    dpos = torch.from_numpy(pos).to(gpu_device)
    out = torch.full_like(dq, float("nan"))
    lse = torch.full((m, hq), float("nan"), device=gpu_device)
    if chunk:
        api.pkv_chunk_attn(cfg, dq, dk, dv, dpos, out, chunk)
    else:
        api.pkv_sparse_row_attn(cfg, dq, dk, dv, dpos, out, lse)
    got, q, k, v = host(out), *(t.astype(np.float64) for t in (q, k, v))
    for a in range(0, m, chunk or m):
        b = min(m, a + (chunk or m))
        keys = slice(a, b) if chunk else slice(None)
        want, want_lse = O.sparse_row_attn(q[a:b], k[keys], v[keys], pos[a:b], dtype="f32")
        assert rel_err(got[a:b], want) <= BAR
        if not chunk:
            assert np.abs(host(lse) - want_lse).max() <= BAR * max(1.0, np.abs(want_lse).max())
