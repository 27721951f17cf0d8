"""GPU parity of the bf16 projection and linear kernels on each of their tiles (64, 128, 192 and
256 tokens high), with one row, at and around the tiles' edges, with and without splits of the
contraction, and with as few and odd steps of it as a tile takes.

Bar: bf16 has 8 significant bits, so a rounding moves a value by at most 2^-8 of it, and an
intermediate whose fp32 sum falls on the other side of a tie ends one unit, at most 2^-7, away.
The sum itself is off by a few times sqrt(n) 2^-24 of its absolute terms: with unit-scale outputs
and n <= 5120 less than 1e-4 of the largest output."""

import numpy as np
import pytest
import torch

from paper_2602_02579_amd import api

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -7

# rows, inputs, features: the tile that the rule takes and its splits of the contraction
SHAPES = [
    (1, 320, 512),        # 64 x 1, five steps
    (64, 1024, 2048),     # 64
    (65, 512, 768),       # 64, one row in the last tile
    (385, 4096, 1024),    # 64 x 4
    (600, 4096, 4096),    # 128
    (129, 4096, 6144),    # 128 x 2, one row in the last tile
    (1300, 512, 6144),    # 192
    (1729, 4096, 6144),   # 192, one row in the last tile
    (883, 5120, 5120),    # 192 x 2
    (961, 256, 12288),    # 256, four steps
    (300, 160, 512),      # 256, contraction no multiple of 64
    (769, 256, 28672),    # 512 rows on 256-token tiles, 257 on 192-token ones, in one launch
    (1921, 256, 12288),   # 1280 and 641
]


def draw(device, seed, *shape, scale=1.0):
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    return (torch.randn(shape, generator=gen, device=device) * scale).bfloat16()


def within(got, want, bound):
    err = (got.double() - want).abs()
    bad = err > bound + 1e-4 * want.abs().max()
    assert not bad.any(), f"{int(bad.sum())} off, worst {err[bad].max().item():.3g}"


def product(x, w):
    return x.double() @ w.double().t()


@pytest.mark.parametrize("m,k,n", SHAPES)
def test_linear_with_residual_in_place(gpu_device, m, k, n):
    x, w = draw(gpu_device, 1, m, k), draw(gpu_device, 2, n, k, scale=k ** -0.5)
    y = draw(gpu_device, 3, m + 1, n)
    guard = y[m].clone()
    res = y[:m].double()
    ws = torch.empty(max(256, api.pkv_glue_workspace_bytes(torch.bfloat16, m, k, n)),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_linear_rows(x, w, y[:m], y[:m], ws=ws)
    p = product(x, w)
    want = p.bfloat16().double() + res
    within(y[:m], want, ULP * (p.abs() + 0.5 * want.abs()))
    assert torch.equal(y[m], guard)


@pytest.mark.parametrize("m,k,n", SHAPES)
def test_gated(gpu_device, m, k, n):
    x = draw(gpu_device, 1, m, k)
    wg, wu = (draw(gpu_device, s, n // 2, k, scale=k ** -0.5) for s in (2, 3))
    y = torch.zeros((m + 1, n // 2), dtype=torch.bfloat16, device=gpu_device)
    ws = torch.empty(max(256, api.pkv_glue_workspace_bytes(torch.bfloat16, m, k, n // 2)),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_swiglu_rows(x, wg, wu, y[:m], ws=ws)
    a, b = (product(x, w).bfloat16().double() for w in (wg, wu))
    want = (a * torch.sigmoid(a)).bfloat16().double() * b
    # silu' <= 1.1: a gate one unit away moves the result by at most 1.1 units of a b; silu and
    # up by a unit each, the last rounding by half of one
    within(y[:m], want, ULP * (1.1 * (a * b).abs() + 2.5 * want.abs()))
    assert not y[m].any()


@pytest.mark.parametrize("variant", ["plain", "bias", "norm"])
@pytest.mark.parametrize("m,k,n", SHAPES)
def test_projection(gpu_device, m, k, n, variant):
    d, theta, eps = 128, 5e5, 1e-5
    hkv = 2
    hq = n // d - 2 * hkv
    if hq < 2:
        hq, hkv = 2, 2
    cfg = api.LayerCfg(hq, hkv, d, k, theta, "bf16")
    hidden = draw(gpu_device, 1, m + 7, k)
    ws_ = [draw(gpu_device, 2 + i, h * d, k, scale=k ** -0.5) for i, h in enumerate((hq, hkv, hkv))]
    rows = torch.from_numpy(np.sort(np.random.default_rng(m).choice(m + 7, m, replace=False))
                            .astype(np.int32)).to(gpu_device)
    pos = rows * 31 + 2
    kw = {}
    if variant == "bias":
        kw = {b: draw(gpu_device, 6 + i, h * d) for i, (b, h) in
              enumerate((("bq", hq), ("bk", hkv), ("bv", hkv)))}
    elif variant == "norm":
        kw = {g: (1 + draw(gpu_device, 9 + i, d, scale=0.2).float()).bfloat16()
              for i, g in enumerate(("q_norm", "k_norm"))}
        kw["norm_eps"] = eps
    ws = torch.empty(max(256, api.pkv_workspace_bytes(api.CALL_GATHER_QKV_PROJ, cfg, 0, m)),
                     dtype=torch.uint8, device=gpu_device)
    q = torch.empty((m, hq, d), dtype=torch.bfloat16, device=gpu_device)
    kc = torch.zeros((m + 7, hkv, d), dtype=torch.bfloat16, device=gpu_device)
    vc = torch.zeros_like(kc)
    if variant == "plain":
        k_out, v_out = torch.empty_like(kc[:m]), torch.empty_like(vc[:m])
        api.pkv_gather_qkv_proj(cfg, hidden, rows, pos, *ws_, q, k_out, v_out, ws=ws)
        kc[rows.long()], vc[rows.long()] = k_out, v_out
    else:
        api.pkv_gather_qkv_proj_scatter(cfg, hidden, rows, pos, *ws_, q, kc, vc, rows, ws=ws, **kw)
    x = hidden[rows.long()]
    ang = pos.double()[:, None] * theta ** (
        -torch.arange(0, d, 2, device=gpu_device, dtype=torch.float64) / d)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    for got, w, bias, gain, heads in ((q, ws_[0], "bq", "q_norm", hq),
                                      (kc[rows.long()], ws_[1], "bk", "k_norm", hkv),
                                      (vc[rows.long()], ws_[2], "bv", None, hkv)):
        y = product(x, w)
        if bias in kw:
            y = y + kw[bias].double()
        y = y.view(m, heads, d)
        if gain in kw:
            y = y * torch.rsqrt(y.square().mean(-1, keepdim=True) + eps) * kw[gain].double()
        if bias != "bv":
            a, b = y[..., :d // 2], y[..., d // 2:]
            y = torch.cat([a * c - b * s, b * c + a * s], -1)
        within(got, y, 0.5 * ULP * y.abs())
    rest = torch.ones(m + 7, dtype=torch.bool, device=gpu_device)
    rest[rows.long()] = False
    assert not kc[rest].any() and not vc[rest].any()
