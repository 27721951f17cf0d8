"""GPU parity of the fp32 matrix-core kernels at the edges of their tiles: 64-row, 16-row and 32-column
(16-pair) tiles and 128-wide contraction chunks of the projection and the linear layers, 16-key
tiles and 16-column tiles of score and attention, fewer keys than waves, ranges of keys.

Bar: a sum of n fp32 products differs from the exact one by at most about n units of 2^-24 of its
absolute sum, whatever the order; n <= 520 here, so 520 * 6e-8 = 3.1e-5 of the largest output
(exponentials and square roots add a few units of 2^-24 of their own)."""

import numpy as np
import pytest
import torch

from oracle import pkv_model_oracle as MO
from oracle import pkv_oracle as O
from paper_2602_02579_amd import api
from tests.test_gpu_kernels import dev, host, lcfg, rel_err, rnd

pytestmark = pytest.mark.gpu

BAR = 3.2e-5


@pytest.mark.parametrize("m,hq,hkv,d,hid", [
    (1, 1, 1, 16, 8), (63, 3, 1, 48, 120), (64, 4, 2, 32, 128), (65, 2, 2, 64, 136),
    (130, 5, 5, 128, 520)])
def test_projection(gpu_device, m, hq, hkv, d, hid):
    cfg = lcfg("f32", hq, hkv, d, hid, 10000.0)
    hidden = rnd(1, (m + 9, hid), "f32")
    wq, wk, wv = (rnd(2 + i, (h * d, hid), "f32", hid ** -0.5) for i, h in enumerate((hq, hkv, hkv)))
    bias = [rnd(6 + i, (h * d,), "f32", 0.5) for i, h in enumerate((hq, hkv, hkv))]
    rows = np.sort(np.random.default_rng(m).choice(m + 9, m, replace=False)).astype(np.int32)
    pos = (rows * 31 + 2).astype(np.int32)
    args = [dev(x, "f32", gpu_device) for x in (hidden, wq, wk, wv)]
    r, p = torch.from_numpy(rows).to(gpu_device), torch.from_numpy(pos).to(gpu_device)
    q = torch.empty((m, hq, d), device=gpu_device)
    kc = torch.zeros((m + 9, hkv, d), device=gpu_device)
    vc = torch.zeros_like(kc)
    api.pkv_gather_qkv_proj_scatter(cfg, args[0], r, p, *args[1:], q, kc, vc, r,
                                    bq=dev(bias[0], "f32", gpu_device),
                                    bk=dev(bias[1], "f32", gpu_device),
                                    bv=dev(bias[2], "f32", gpu_device))
    x = hidden.astype(np.float64)[rows]
    want = []
    for w, b, h in ((wq, bias[0], hq), (wk, bias[1], hkv), (wv, bias[2], hkv)):
        want.append((x @ w.astype(np.float64).T + b).reshape(m, h, d))
    assert rel_err(host(q), O.rope_rotate(want[0], pos, 10000.0)) <= BAR
    assert rel_err(host(kc)[rows], O.rope_rotate(want[1], pos, 10000.0)) <= BAR
    assert rel_err(host(vc)[rows], want[2]) <= BAR
    rest = np.setdiff1d(np.arange(m + 9), rows)
    assert not host(kc)[rest].any() and not host(vc)[rest].any()


# the first five are little work and take a wave per output, the next four tiles of 16 rows, the
# last three tiles of 64
@pytest.mark.parametrize("m,k,n", [(1, 8, 8), (63, 128, 24), (65, 136, 40), (64, 256, 72),
                                   (17, 520, 104), (130, 8, 72), (97, 24, 520), (64, 128, 264),
                                   (321, 136, 200), (1025, 24, 520), (1088, 128, 512),
                                   (1100, 520, 504)])
def test_linear_layers(gpu_device, m, k, n):
    x, w, u = rnd(1, (m, k), "f32"), rnd(2, (n, k), "f32", k ** -0.5), rnd(3, (n, k), "f32", k ** -0.5)
    res = rnd(4, (m, n), "f32")
    dx, dw, du, y = (dev(t, "f32", gpu_device) for t in (x, w, u, res))
    api.pkv_linear_rows(dx, dw, y, y)                       # in place, as the carried rows use it
    f = [t.astype(np.float64) for t in (x, w, u, res)]
    assert rel_err(host(y), MO.linear_rows(f[0], f[1], f[3], "f32")) <= BAR
    api.pkv_swiglu_rows(dx, dw, du, y)
    assert rel_err(host(y), MO.swiglu_up(f[0], f[1], f[2], "f32")) <= BAR


@pytest.mark.parametrize("nq,n_ctx,hq,hkv,d", [
    (1, 1, 1, 1, 32), (1, 17, 4, 4, 64), (5, 63, 6, 2, 32), (16, 65, 4, 4, 64), (33, 520, 8, 2, 128)])
def test_score_and_attention(gpu_device, nq, n_ctx, hq, hkv, d):
    cfg = lcfg("f32", hq, hkv, d)
    q, k, v = rnd(1, (nq, hq, d), "f32"), rnd(2, (n_ctx, hkv, d), "f32"), rnd(3, (n_ctx, hkv, d), "f32")
    dq, dk, dv = (dev(t, "f32", gpu_device) for t in (q, k, v))
    ws = torch.full((max(api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, cfg, n_ctx, nq), 256),), 0xff,
                    dtype=torch.uint8, device=gpu_device)
    score = torch.empty(n_ctx, device=gpu_device)
    api.pkv_query_score(cfg, dq, dk, score, ws=ws)
    q64, k64 = q.astype(np.float64), k.astype(np.float64)
    want = O.query_score(q64, k64)
    assert rel_err(host(score), want) <= BAR
    pos = np.sort(np.random.default_rng(nq).integers(0, n_ctx, nq)).astype(np.int32)
    pos[-1] = n_ctx - 1
    out = torch.empty_like(dq)
    lse = torch.empty((nq, hq), device=gpu_device)
    api.pkv_sparse_row_attn(cfg, dq, dk, dv, torch.from_numpy(pos).to(gpu_device), out, lse)
    w_out, w_lse = O.sparse_row_attn(q64, k64, v.astype(np.float64), pos, dtype="f32")
    assert rel_err(host(out), w_out) <= BAR
    assert np.abs(host(lse) - w_lse).max() <= BAR * max(1.0, np.abs(w_lse).max())
    # given normalisers, each row counting for the keys it sees: columns of the same attention
    api.pkv_query_score_lse(cfg, dq, dk, lse, torch.from_numpy(pos).to(gpu_device), score, ws=ws)
    s = np.einsum("qhd,thd->qht", q64, np.repeat(k64, hq // hkv, 1)) * d ** -0.5
    p = np.exp(s - w_lse[:, :, None]) * (np.arange(n_ctx)[None, None] <= pos[:, None, None])
    assert rel_err(host(score), p.sum((0, 1)) / (nq * hq)) <= BAR
