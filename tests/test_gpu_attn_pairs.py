"""GPU parity of the attention whose jobs are 128 columns with the keys shared by two groups of waves
(contexts of a few thousand keys): row limits at the edges of its 32-key blocks and of the pairs of
them, caches that end inside a block, groups whose rows do not fill the columns, rows in any order, rows
that see a single key, scores that keep growing (the second attempt), and, at the counts of jobs and
keys where the launch goes to it and where it no longer does, that it does."""

import numpy as np
import pytest
import torch

from paper_2602_02579_amd import api, synth
from tests.test_gpu_attn_short_ranges import check
from tests.test_gpu_kernels import TOL, lcfg, rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("growing", [False, True])
@pytest.mark.parametrize("m,n_keys,hq,hkv,order,pairs", [
    (200, 1120, 32, 8, "sorted", True),      # 56 jobs: as few as 1120 keys take
    (200, 1121, 32, 8, "sorted", False),     # a key too many
    (1030, 1030, 40, 8, "sorted", True),     # 336 jobs, 125 of 128 columns
    (1024, 1040, 32, 8, "sorted", True),     # 256 jobs
    (700, 1503, 35, 5, "any", True),         # groups of seven heads, cache ends inside a block
    (400, 1217, 16, 16, "any", True),        # groups of one: 128 rows a job
    (100, 1089, 64, 8, "end", True)])
def test_pairs(gpu_device, m, n_keys, hq, hkv, order, pairs, growing):
    assert (api.pkv_sparse_row_attn_kernel(lcfg("bf16", hq, hkv, 128), n_keys, m)
            == api.ATTN_PAIRS) == pairs
    q, vc = rnd(1, (m, hq, 128), "bf16"), rnd(3, (n_keys, hkv, 128), "bf16")
    kc = rnd(2, (n_keys, hkv, 128), "bf16")
    if growing:   # up to ~60 nats between the first and the last key
        kc = synth.to_storage(kc * np.linspace(0.05, 5.0, n_keys, dtype=np.float32)[:, None, None],
                              "bf16")
    gen = np.random.default_rng(m)
    if order == "end":
        pos = np.arange(n_keys - m, n_keys)
    else:
        pos = gen.choice(n_keys, m, replace=False)
        edges = [0, 1, 30, 31, 32, 33, 62, 63, 64, 65, 95, 96, 127, 128, 129, n_keys - 1]
        pos[:len(edges)] = edges
        if order == "sorted":
            pos.sort()
    check(gpu_device, hq, hkv, q, kc, vc, pos.astype(np.int32))


@pytest.mark.parametrize("m,n_keys,hq,hkv,pairs", [
    (2560, 2611, 32, 8, True), (2561, 2611, 32, 8, False),      # 640 jobs, and 648
    (2000, 12288, 32, 8, True), (2000, 12289, 32, 8, False),
    (1600, 3001, 40, 8, True), (1632, 3001, 40, 8, False)])     # 512 jobs, and 528 on 256 CUs
def test_most_jobs_and_keys(gpu_device, m, n_keys, hq, hkv, pairs):
    """Against the fp64 attention on the device, head by head."""
    cfg = lcfg("bf16", hq, hkv, 128)
    assert (api.pkv_sparse_row_attn_kernel(cfg, n_keys, m) == api.ATTN_PAIRS) == pairs
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(m + n_keys)
    q, k, v = (torch.randn(s, generator=gen, device=gpu_device).to(torch.bfloat16)
               for s in ((m, hq, 128), (n_keys, hkv, 128), (n_keys, hkv, 128)))
    pos = torch.randperm(n_keys, generator=gen, device=gpu_device)[:m].sort()[0].to(torch.int32)
    pos[0], pos[-1] = 0, n_keys - 1
    out = torch.full_like(q, float("nan"))
    ws = torch.empty(max(256, api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m)),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_sparse_row_attn(cfg, q, k, v, pos, out, None, ws=ws)
    hidden = torch.arange(n_keys, device=gpu_device) > pos[:, None]
    for h in range(0, hq, 3):
        g = h // (hq // hkv)
        s = q[:, h].double() @ k[:, g].double().t() * 128 ** -0.5
        want = torch.softmax(s.masked_fill_(hidden, float("-inf")), -1) @ v[:, g].double()
        err = (out[:, h].double() - want).abs().max() / want.abs().max()
        assert err <= TOL["bf16"], (h, err)
