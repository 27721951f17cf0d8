"""fp32 decoder layers whose projection and gated layer normalise the rows themselves: against the fp64
oracle over several chunks of the contraction, the last one ragged, row tiles that the rows do not
fill, and at the edges of the rule - the longest rows that are normalised inside a launch, the most
tiles that run at once, and one step beyond, where the normalisation is a launch of its own (and
writes x).

Bar: a sum of n fp32 products is off by at most about n units of 2^-24 of its absolute sum, the
normalisation by the order of its n squares (n / 32 in a chain, then a tree): n + 32 in all."""

import numpy as np
import pytest
import torch

from oracle import pkv_model_oracle as MO
from oracle import pkv_oracle as O
from paper_2602_02579_amd import api
from tests.test_gpu_kernels import dev, host, lcfg, rel_err, rnd

pytestmark = pytest.mark.gpu

EPS, UNTOUCHED = 1e-5, 7.0


def bar(n):
    return (n + 32) * 2.0 ** -24


def layer(gpu_device, m, hid, hq, hkv, d, inter, bias=False):
    gain = lambda s: 1.0 + rnd(s, (hid,), "f32", 0.1)   # noqa: E731
    L = dict(w_in=gain(1), w_post=gain(2))
    for s, (name, rows, cols) in enumerate((
            ("wq", hq * d, hid), ("wk", hkv * d, hid), ("wv", hkv * d, hid), ("wo", hid, hq * d),
            ("w_gate", inter, hid), ("w_up", inter, hid), ("w_down", hid, inter))):
        L[name] = rnd(3 + s, (rows, cols), "f32", cols ** -0.5)
    if bias:
        L.update(bq=rnd(20, (hq * d,), "f32"), bk=rnd(21, (hkv * d,), "f32"),
                 bv=rnd(22, (hkv * d,), "f32"))
    L["w_down"][:] = 0.0          # so that h ends as the gated layer's input
    h = rnd(30, (m, hid), "f32")
    D = {k: dev(v, "f32", gpu_device) for k, v in L.items()}
    new = lambda *s: torch.full((m + 1,) + s, UNTOUCHED, device=gpu_device)   # noqa: E731
    b = dict(h=new(hid), x=new(hid), q=new(hq, d), attn=new(hq, d), g=new(inter))
    b["h"][:m] = dev(h, "f32", gpu_device)
    b["k"], b["v"] = (torch.zeros((m, hkv, d), device=gpu_device) for _ in range(2))
    return L, D, h, b


def run(gpu_device, cfg, D, b, m, dst, stop):
    pos = torch.arange(m, dtype=torch.int32, device=gpu_device)
    api.pkv_layer_rows(cfg, b["h"], b["x"], b["q"], b["attn"], b["g"], m, D, ("bq", "bk", "bv"),
                       b["k"], b["v"], pos, dst, EPS, torch.empty(256, dtype=torch.uint8,
                                                                   device=gpu_device),
                       chunk_len=m, stop=stop)
    for name in ("h", "x", "q", "attn", "g"):
        assert (b[name][m] == UNTOUCHED).all(), name   # the row behind the last


@pytest.mark.parametrize("m,hid,hq,hkv,d,inside", [
    (5, 8, 1, 1, 32, True), (33, 136, 4, 2, 64, True), (21, 264, 3, 3, 48, True),
    (672, 256, 4, 4, 64, True), (673, 256, 4, 4, 64, False),     # 42 and 43 x 24 tiles
    (96, 640, 32, 16, 64, True), (97, 640, 32, 16, 64, False),   # 6 and 7 x 128
    (37, 768, 2, 2, 32, True), (37, 776, 2, 2, 32, False), (1100, 136, 8, 4, 64, False)])
@pytest.mark.parametrize("with_q", [True, False])
def test_projection(gpu_device, m, hid, hq, hkv, d, inside, with_q):
    cfg = lcfg("f32", hq, hkv, d, hid, 1e4)
    L, D, h, b = layer(gpu_device, m, hid, hq, hkv, d, 8, bias=hid == 136)
    order = np.random.default_rng(m).permutation(m).astype(np.int32)
    dst = torch.from_numpy(order).to(gpu_device)
    # tiles are fewer without Q: the row counts above are edges of the whole projection
    fused = inside
    if not with_q:
        columns = 2 * -(-hkv * d // 32)
        low, high = -(-m // 16) * columns, -(-m // 64) * columns
        fused = hid <= 768 and (low <= 768 or (low <= 1024 and high > 256))
    run(gpu_device, cfg, D, b, m, dst, api.LAYER_TO_SCORES if with_q else api.LAYER_TO_CACHES)
    x = MO.rmsnorm_rows(h, None, L["w_in"], EPS, "f64")
    pos = np.arange(m)
    for name, w, c, heads, rows in (("q", "wq", "bq", hq, pos), ("k", "wk", "bk", hkv, order),
                                    ("v", "wv", "bv", hkv, order)):
        if name == "q" and not with_q:
            assert (b["q"] == UNTOUCHED).all()
            continue
        want = x @ L[w].astype(np.float64).T + (L[c].astype(np.float64) if c in L else 0.0)
        want = want.reshape(m, heads, d)
        want = want if name == "v" else O.rope_rotate(want, pos, 1e4)
        assert rel_err(host(b[name])[rows], want) <= bar(hid), name
    assert bool((b["x"] == UNTOUCHED).all()) == fused
    if not fused:
        assert rel_err(host(b["x"][:m]), x) <= bar(hid)


@pytest.mark.parametrize("m,hid,inter,inside", [
    (1, 8, 8, True), (33, 136, 200, True), (150, 256, 520, True),
    (512, 256, 512, True), (513, 256, 512, False),                # 32 and 33 x 32 tiles
    (40, 384, 264, True), (40, 392, 264, False), (17, 640, 72, False)])
def test_gated_layer(gpu_device, m, hid, inter, inside):
    cfg = lcfg("f32", 1, 1, 32, hid, 1e4)
    L, D, h, b = layer(gpu_device, m, hid, 1, 1, 32, inter)
    dst = torch.arange(m, dtype=torch.int32, device=gpu_device)
    run(gpu_device, cfg, D, b, m, dst, api.LAYER_WHOLE)
    y = MO.rmsnorm_rows(host(b["h"])[:m], None, L["w_post"], EPS, "f64")
    gate, up = (y @ L[w].astype(np.float64).T for w in ("w_gate", "w_up"))
    want = gate / (1.0 + np.exp(-gate)) * up
    # the slope of silu is at most 1.1
    assert np.abs(host(b["g"])[:m] - want).max() <= (
        2.1 * bar(hid) * np.abs(gate).max() * np.abs(up).max())
    assert bool((b["x"] == UNTOUCHED).all()) == inside     # (these rows' projection never writes x)
    if not inside:
        assert rel_err(host(b["x"][:m]), y) <= bar(hid)
