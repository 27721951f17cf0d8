"""GPU parity of the attention where the keys of a row tile run in ranges of a few 64-key
steps (the fewest there are: two), with ordinary scores and with late ones far above the first
keys of a range, which make the job of that range run a second time with its columns' true
maxima; and of launches just below and just above one job per compute unit, where the work
queue comes in.

Caches of up to 768 keys take a kernel without ranges at launches this small, unless a
transposed copy of the values is asked for: every shape runs with each source of the values."""

import numpy as np
import pytest
import torch

from oracle import pkv_oracle as O
from paper_2602_02579_amd import api, synth
from tests.test_gpu_kernels import TOL, dev, host, lcfg, rel_err, rnd

pytestmark = pytest.mark.gpu


def check(gpu_device, hq, hkv, q, kc, vc, pos):
    cfg = lcfg("bf16", hq, hkv, 128)
    m, n_keys = len(pos), kc.shape[0]
    want, want_lse = O.sparse_row_attn(q.astype(np.float64), kc.astype(np.float64),
                                       vc.astype(np.float64), pos, dtype="bf16")
    out = torch.empty((m, hq, 128), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.empty((m, hq), dtype=torch.float32, device=gpu_device)
    ws = torch.full((max(api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m), 256),),
                    0xff, dtype=torch.uint8, device=gpu_device)
    api.pkv_sparse_row_attn(cfg, dev(q, "bf16", gpu_device), dev(kc, "bf16", gpu_device),
                            dev(vc, "bf16", gpu_device), torch.from_numpy(pos).to(gpu_device),
                            out, lse, ws=ws)
    got, got_lse = host(out), host(lse)
    assert np.isfinite(got).all() and np.isfinite(got_lse).all()
    assert rel_err(got, want) <= TOL["bf16"]
    # as in the full-size tests: 4e-3 where the normaliser is of order ten or less
    assert np.abs(got_lse - want_lse).max() <= 4e-3 * max(1.0, np.abs(want_lse).max() / 10)


def planned_ranges(cfg, n_keys, m):
    """Ranges that the keys of a row tile are cut into: the workspace holds V^T, one counter per
    kv head (both rounded up to 256 bytes) and, with more than one range, an fp32 output row and
    its log-sum-exp per (range, row, head)."""
    def up(x, to):
        return (x + to - 1) // to * to
    fixed = up(cfg.n_kv_heads * cfg.head_dim * up(n_keys, 64) * 2, 256) + up(4 * cfg.n_kv_heads, 256)
    rest = api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m) - fixed
    return max(1, rest // (m * cfg.n_q_heads * (cfg.head_dim + 1) * 4))


@pytest.mark.parametrize("late", [False, True])
@pytest.mark.parametrize("m,n_keys,ranges,length", [
    (1, 255, 1, 256), (1, 256, 1, 256), (3, 257, 1, 320), (5, 385, 3, 192), (65, 449, 3, 192),
    (17, 2049, 11, 192), (1, 769, 5, 192), (1, 1536, 12, 128), (5, 896, 7, 128),
    (33, 1280, 10, 128), (65, 384, 3, 128)])
def test_short_ranges(gpu_device, v_source, m, n_keys, ranges, length, late):
    hq, hkv = 8, 2
    assert planned_ranges(lcfg("bf16", hq, hkv, 128), n_keys, m) == ranges
    assert ranges == 1 or -(-n_keys // ranges) <= length < -(-n_keys // ranges) + 64
    g = np.random.default_rng(100 + m + n_keys)
    q, vc = rnd(1, (m, hq, 128), "bf16"), rnd(3, (n_keys, hkv, 128), "bf16")
    kc = rnd(2, (n_keys, hkv, 128), "bf16", 0.05 if late else 1.0)
    if late:   # ~180 nats above the first 32 keys of every range, which give its reference
        q[m // 2:, 1] = 4.0
        for start in range(0, n_keys, length):
            kc[start + 40:start + 90:9, 0] = 4.0
        q, kc = synth.to_storage(q, "bf16"), synth.to_storage(kc, "bf16")
    pos = np.sort(g.choice(n_keys, m, replace=False)).astype(np.int32)
    pos[-1] = n_keys - 1
    check(gpu_device, hq, hkv, q, kc, vc, pos)


@pytest.mark.parametrize("m", [64 * 32, 64 * 32 + 1])   # 256 and 264 jobs over 8 kv heads
def test_one_job_per_cu_and_one_row_more(gpu_device, m):
    hq, hkv, n_keys = 32, 8, 200
    g = np.random.default_rng(m)
    pos = np.sort(g.integers(0, n_keys, m)).astype(np.int32)
    check(gpu_device, hq, hkv, rnd(4, (m, hq, 128), "bf16"), rnd(5, (n_keys, hkv, 128), "bf16"),
          rnd(6, (n_keys, hkv, 128), "bf16"), pos)
