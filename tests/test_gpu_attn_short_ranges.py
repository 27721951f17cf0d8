"""GPU parity of the attention where the keys of a row tile run in ranges of a few 64-key
steps (the fewest there are: two), with ordinary scores and with late ones far above the first
keys of a range, which make the job of that range run a second time with its columns' true
maxima; and of launches just below and just above one job per compute unit, where the work
queue comes in."""

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


@pytest.mark.parametrize("late", [False, True])
@pytest.mark.parametrize("m,n_keys", [(1, 255), (1, 256), (3, 257), (5, 385), (65, 449), (17, 2049)])
def test_short_ranges(gpu_device, m, n_keys, late):
    hq, hkv = 8, 2
    g = np.random.default_rng(100 + m + n_keys)
    q, vc = rnd(1, (m, hq, 128), "bf16"), rnd(3, (n_keys, hkv, 128), "bf16")
    kc = rnd(2, (n_keys, hkv, 128), "bf16", 0.05 if late else 1.0)
    if late:   # ~180 nats above the first keys of every range from the second one on
        q[m // 2:, 1] = 4.0
        kc[200::37, 0] = 4.0
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
