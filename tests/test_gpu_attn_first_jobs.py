"""Attention with a work queue: every job is done once, however the first ones are handed out - by the
workgroups' numbers or claimed - with kv heads that divide the workgroups and that do not, one job
more than there are compute units, several jobs each, and one to three ranges of the keys."""

import pytest
import torch

from paper_2602_02579_amd import api
from tests.test_gpu_attn_short_ranges import planned_ranges
from tests.test_gpu_kernels import TOL, lcfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,m,n_keys,ranges", [
    (16, 1, 4100, 300, 1), (16, 1, 1373, 3100, 3),   # 257 jobs of one head, and 258 of three ranges
    (48, 3, 1376, 700, 1), (48, 3, 685, 2800, 2),    # 258 jobs of three heads
    (35, 5, 1880, 500, 1), (56, 7, 1180, 400, 1), (56, 7, 3000, 400, 1),
    (32, 2, 2060, 400, 1), (32, 2, 1037, 2500, 2), (32, 2, 1037, 3100, 3),
    (28, 4, 1185, 2500, 2), (28, 4, 789, 3100, 3), (64, 4, 3000, 500, 1),
    (128, 8, 600, 300, 1), (128, 8, 2100, 300, 1)])
@pytest.mark.parametrize("source", ["0", "1"])
def test_every_job_is_done(gpu_device, monkeypatch, hq, hkv, m, n_keys, ranges, source):
    monkeypatch.setenv("PKV_ATTN_VT", "1")       # where the values come from decides the kernel, too
    cfg = lcfg("bf16", hq, hkv, 128)
    assert planned_ranges(cfg, n_keys, m) == ranges
    assert api.pkv_sparse_row_attn_kernel(cfg, n_keys, m) == api.ATTN_QUEUE
    monkeypatch.setenv("PKV_ATTN_VT", source)    # (values as they are: pairs take some of the sizes)
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(m + n_keys)
    q, k, v = (torch.randn(s, generator=gen, device=gpu_device).to(torch.bfloat16)
               for s in ((m, hq, 128), (n_keys, hkv, 128), (n_keys, hkv, 128)))
    pos = torch.randint(0, n_keys, (m,), generator=gen, device=gpu_device).sort()[0].to(torch.int32)
    pos[0], pos[-1] = 0, n_keys - 1
    out = torch.full_like(q, float("nan"))
    ws = torch.full((max(256, api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m)),),
                    255, dtype=torch.uint8, device=gpu_device)
    api.pkv_sparse_row_attn(cfg, q, k, v, pos, out, None, ws=ws)
    hidden = torch.arange(n_keys, device=gpu_device) > pos[:, None]
    for h in range(hq):                          # against the fp64 attention, head by head
        g = h // (hq // hkv)
        s = q[:, h].double() @ k[:, g].double().t() * 128 ** -0.5
        want = torch.softmax(s.masked_fill_(hidden, float("-inf")), -1) @ v[:, g].double()
        err = (out[:, h].double() - want).abs().max() / want.abs().max()
        assert err <= TOL["bf16"], (h, err)
