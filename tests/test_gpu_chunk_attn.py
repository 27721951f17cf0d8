"""GPU parity of the attention of many chunks in one call, against the fp64 attention of every chunk
by itself: both kernels that take the chunks by a grid and the geometries that go chunk by chunk,
last chunks of a full tile, one row more and one row, chunks at and above the limit of the shared
launch, and a single chunk; and of the chunk producer when its chunks fill more than one group."""

import numpy as np
import pytest
import torch

from oracle import pkv_oracle as O
from paper_2602_02579_amd import api, diagnostics
from tests.test_gpu_diagnostics import make_model, to_dev
from tests.test_gpu_kernels import rnd
from tests.test_gpu_model import CASES, EPS

pytestmark = pytest.mark.gpu

TDT = {"f32": torch.float32, "bf16": torch.bfloat16}


@pytest.mark.parametrize("dtype,hq,hkv,d,m,chunk_len", [
    ("bf16", 8, 2, 128, 300, 128),      # last chunk of 44
    ("bf16", 8, 2, 128, 257, 64),       # last chunk of one row
    ("bf16", 10, 2, 128, 130, 65),      # 25 rows per job; chunks of a tile and a row
    ("bf16", 32, 8, 128, 2048, 1024),   # two jobs per compute unit, the longest chunk
    ("bf16", 4, 2, 128, 2100, 1025),    # too long for the shared launch
    ("bf16", 8, 2, 128, 100, 128),      # one chunk
    ("bf16", 8, 2, 64, 200, 96),        # chunk by chunk
    ("f32", 4, 4, 64, 1000, 333), ("f32", 8, 2, 128, 131, 130), ("f32", 4, 2, 32, 70, 16),
    ("f32", 2, 2, 48, 50, 20)])         # chunk by chunk
def test_chunks_attend_within_themselves(gpu_device, dtype, hq, hkv, d, m, chunk_len):
    q, k, v = rnd(1, (m, hq, d), dtype), rnd(2, (m, hkv, d), dtype), rnd(3, (m, hkv, d), dtype)
    cfg = api.LayerCfg(hq, hkv, d, 64, 1e4, dtype)
    dq, dk, dv = (torch.from_numpy(x).to(TDT[dtype]).to(gpu_device) for x in (q, k, v))
    pos = np.arange(m, dtype=np.int32) % chunk_len
    out = torch.full_like(dq, float("nan"))
    ws = torch.empty(max(256, api.pkv_chunk_attn_workspace_bytes(cfg, m, chunk_len)),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_chunk_attn(cfg, dq, dk, dv, torch.from_numpy(pos).to(gpu_device), out, chunk_len, ws=ws)
    got = out.cpu().double().numpy()
    # one rounding of the output and, bf16, one of the probabilities; fp32 sums
    tol = 1e-4 if dtype == "f32" else 2e-2
    for a in range(0, m, chunk_len):
        b = min(m, a + chunk_len)
        want, _ = O.sparse_row_attn(*(x[a:b].astype(np.float64) for x in (q, k, v)), pos[a:b],
                                    dtype=dtype)
        assert np.abs(got[a:b] - want).max() <= tol * np.abs(want).max(), (a, b)


@pytest.mark.parametrize("name", ["f32-small", "bf16-tiles"])
def test_groups_of_chunks_are_the_chunks(gpu_device, name, monkeypatch):
    """Chunks that pass together give what they give one by one, up to the order of the sums that the
    tiles of another row count choose: fp32, three layers of sums of at most 160 products, each off by
    as many units of 2^-24; bf16, the tolerance of the chunk caches' parity test."""
    cfg, inter = CASES[name]
    embed, blocks = to_dev(cfg, *make_model(cfg, inter), gpu_device)
    got = []
    for rows in (64, 1):     # groups of two chunks; every chunk a group of its own
        monkeypatch.setattr(diagnostics, "GROUP_ROWS", rows)
        got.append(diagnostics.Diagnostics(cfg, inter, EPS, gpu_device).chunk_isolated_cache(
            embed, blocks, 30))
    tol = 3 * 160 * 2.0 ** -24 if cfg.dtype == "f32" else 2e-2
    for a, b in zip(got[0][0] + got[0][1], got[1][0] + got[1][1]):
        a, b = a.double(), b.double()
        assert (a - b).abs().max() <= tol * b.abs().max()
