"""GPU parity of the attention of launches with more jobs than compute units where some jobs are
done twice: scores far above the maximum of a column's first 32 keys (its softmax reference)
take the sums out of their safe range, and the workgroup goes over the job's keys again with the
columns' true maxima before it claims its next job.  Every other row tile and every other kv
head has such scores, so a workgroup's jobs change between one attempt and two; with the values
from the cache as it is and from a transposed copy, with one and with two key ranges."""

import numpy as np
import pytest
import torch

from paper_2602_02579_amd import api
from tests.test_gpu_attn_short_ranges import planned_ranges
from tests.test_gpu_kernels import TOL, lcfg

pytestmark = pytest.mark.gpu


def reference(q, kc, vc, pos):
    """out, lse in fp64, one head at a time"""
    m, hq, d = q.shape
    group = hq // kc.shape[1]
    out = torch.empty((m, hq, d), dtype=torch.float64, device=q.device)
    lse = torch.empty((m, hq), dtype=torch.float64, device=q.device)
    hidden = torch.arange(kc.shape[0], device=q.device)[None] > pos[:, None]
    for h in range(hq):
        s = q[:, h].double() @ kc[:, h // group].double().t().contiguous() * d ** -0.5
        s = s.masked_fill(hidden, float("-inf"))
        lse[:, h] = torch.logsumexp(s, 1)
        out[:, h] = torch.softmax(s, 1) @ vc[:, h // group].double()
    return out, lse


# (m, n_keys, hq, hkv, ranges): 288 jobs of 256 (row, head) columns each; 264; 288 in two ranges
@pytest.mark.parametrize("m,n_keys,hq,hkv,ranges", [(4400, 300, 16, 16, 1), (2049, 500, 32, 8, 1),
                                                    (1100, 3000, 32, 8, 2)])
def test_some_jobs_done_twice(gpu_device, v_source, m, n_keys, hq, hkv, ranges):
    cfg = lcfg("bf16", hq, hkv, 128)
    group, rows_per_tile = hq // hkv, 256 // (hq // hkv)
    assert planned_ranges(cfg, n_keys, m) == ranges
    assert -(-m // rows_per_tile) * hkv * ranges > 256
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(m + n_keys)

    def normal(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=gpu_device) * scale).bfloat16()
    q, kc, vc = normal(m, hq, 128), normal(n_keys, hkv, 128, scale=0.05), normal(n_keys, hkv, 128)
    far = (torch.arange(m, device=gpu_device) // rows_per_tile) % 2 == 1
    for g in range(0, hkv, 2):
        q[far, g * group] = 4.0
        kc[70::97, g] = 4.0            # 16 * 128 / sqrt(128) = 181 nats, 261 bits
    # every range starts with 32 keys none of which is one of those
    length = -(-n_keys // (64 * ranges)) * 64
    for start in range(0, n_keys, length):
        kc[start:start + 32] = normal(min(32, n_keys - start), hkv, 128, scale=0.05)
    rng = np.random.default_rng(m)
    pos = torch.from_numpy(np.sort(rng.integers(0, n_keys, m)).astype(np.int32)).to(gpu_device)
    out = torch.empty((m, hq, 128), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.empty((m, hq), dtype=torch.float32, device=gpu_device)
    ws = torch.full((api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m),), 0xff,
                    dtype=torch.uint8, device=gpu_device)
    want, want_lse = reference(q, kc, vc, pos)
    assert (want_lse[far][:, 0] > 80).any() and (want_lse[~far] < 40).all()
    for _ in range(2):                 # the second pass finds the workspace as the first left it
        out.fill_(float("nan"))
        lse.fill_(float("nan"))
        api.pkv_sparse_row_attn(cfg, q, kc, vc, pos, out, lse, ws=ws)
        err = (out.double() - want).abs().amax(-1)
        assert err.max() <= TOL["bf16"] * want.abs().max()        # NaN fails, too
        # fp32 scores of up to 181 nats, a few units of 2^-24 of it, and exp2 and log of fp32
        assert (lse.double() - want_lse).abs().max() <= 4e-3 * max(
            1.0, want_lse.abs().max().item() / 10)
