"""Attention whose results replace the queries: the bits of the call with an output of its own, on every
kernel - fp32 with head counts that would let several workgroups share a tile of columns, with a
cache and in chunks; bf16 short caches, jobs that share the keys in pairs, key ranges, the work
queue, head_dim 64 and the generic kernel."""

import numpy as np
import pytest
import torch

from paper_2602_02579_amd import api
from tests.test_gpu_kernels import dev, lcfg, rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,m,n_keys,hq,hkv,d,chunk", [
    ("f32", 33, 1040, 4, 4, 64, 0),        # four workgroups would share a tile
    ("f32", 257, 1040, 4, 4, 64, 0),       # two
    ("f32", 64, 700, 8, 2, 128, 0), ("f32", 40, 300, 4, 2, 32, 0), ("f32", 20, 90, 4, 2, 48, 0),
    ("f32", 300, 300, 4, 4, 64, 150), ("f32", 700, 700, 4, 4, 64, 200),
    ("bf16", 300, 300, 8, 2, 128, 130), ("bf16", 200, 700, 8, 2, 128, 0),
    ("bf16", 1030, 1100, 40, 8, 128, 0),   # 336 jobs of 128 columns
    ("bf16", 65, 3000, 8, 2, 128, 0), ("bf16", 775, 5000, 32, 8, 128, 0),
    ("bf16", 2200, 2300, 32, 8, 128, 0), ("bf16", 70, 200, 8, 2, 64, 0),
    ("bf16", 20, 90, 4, 2, 48, 0)])
def test_results_may_replace_the_queries(gpu_device, dtype, m, n_keys, hq, hkv, d, chunk):
    cfg = lcfg(dtype, hq, hkv, d)
    q, k, v = (dev(rnd(s, shape, dtype), dtype, gpu_device) for s, shape in
               ((1, (m, hq, d)), (2, (n_keys, hkv, d)), (3, (n_keys, hkv, d))))
    if chunk:
        pos = np.arange(m, dtype=np.int32) % chunk
        need = api.pkv_chunk_attn_workspace_bytes(cfg, m, chunk)
    else:
        pos = np.sort(np.random.default_rng(m).choice(n_keys, m, replace=False)).astype(np.int32)
        need = api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m)
    pos = torch.from_numpy(pos).to(gpu_device)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device=gpu_device)

    def attend(out):
        if chunk:
            api.pkv_chunk_attn(cfg, q, k, v, pos, out, chunk, ws=ws)
        else:
            api.pkv_sparse_row_attn(cfg, q, k, v, pos, out, None, ws=ws)
    want = torch.empty_like(q)
    attend(want)
    attend(q)
    assert torch.equal(q, want)
