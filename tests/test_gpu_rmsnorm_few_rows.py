"""GPU parity of the RMS norm around the limits of its two kernels: a workgroup per row for up to 2048
rows of 256 to 2048 pieces of 16 bytes and up to 1024 rows of 65 to 255, else a wave per row; one
piece, one more than 256 lanes take, ragged counts, gathered rows.

Bar: the result is rounded once (bf16: 2^-8 of it; a unit, 2^-7, where fp32 falls on the other side
of a tie); fp32: a few units of 2^-24 from the sum over at most 16384 squares of one sign."""

import pytest
import torch

from paper_2602_02579_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gather", [False, True])
@pytest.mark.parametrize("dtype,m,hidden", [
    ("bf16", 1, 8), ("bf16", 3, 2048), ("bf16", 50, 2056), ("bf16", 870, 5120), ("bf16", 33, 16384),
    ("bf16", 1024, 1024), ("bf16", 1025, 1024), ("bf16", 2048, 2048), ("bf16", 2049, 2048),
    ("bf16", 6, 512), ("bf16", 6, 520), ("f32", 7, 8192), ("f32", 7, 8200), ("f32", 70, 64)])
def test_rmsnorm_few_rows(gpu_device, dtype, m, hidden, gather):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(m + hidden)
    h = (3 * torch.randn((m + 5, hidden), generator=gen, device=gpu_device)).to(dt)
    w = (1 + 0.2 * torch.randn(hidden, generator=gen, device=gpu_device)).to(dt)
    rows = torch.randperm(m + 5, generator=gen, device=gpu_device)[:m].int() if gather else None
    y = torch.zeros((m + 1, hidden), dtype=dt, device=gpu_device)
    api.pkv_rmsnorm_rows(h if gather else h[:m], rows, w, 1e-5, y[:m])
    x = (h[rows.long()] if gather else h[:m]).double()
    want = x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5) * w.double()
    bar = 2.0 ** -7 if dtype == "bf16" else 2e-6
    assert ((y[:m].double() - want).abs() <= bar * want.abs()).all()
    assert not y[m].any()
