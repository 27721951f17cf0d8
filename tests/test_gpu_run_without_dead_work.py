"""What a whole run leaves out is not missed: CarriedRows.run (whose last scoring layer stops at its
scores) against stage1 + stage2, and the chunk producer (whose last layer stops at its cache rows)
against a full stage2 over the same rows.  Stage II is the same calls on the same inputs, so with
the same selection every output has the same bits; the selections are the same because the
inputs keep a guard band around the threshold empty."""

import pytest
import torch

from paper_2602_02579_amd import api, diagnostics, model
from tests.test_gpu_model import CASES, EPS, build

pytestmark = pytest.mark.gpu


def setup(name, device):
    cfg, inter = CASES[name]
    embed, layers = build(cfg, inter)
    dev_layers = [model.upload_block(cfg, l, device) for l in layers]
    dt = dev_layers[0]["wq"].dtype
    return cfg, inter, torch.from_numpy(embed).to(dt).to(device), dev_layers


@pytest.mark.parametrize("name", sorted(CASES))
def test_run_is_stage1_and_stage2(gpu_device, name):
    got = []
    for whole in (True, False):
        cfg, inter, embed, layers = setup(name, gpu_device)
        cr = model.CarriedRows(cfg, inter, EPS, gpu_device)
        if whole:
            h = cr.run(embed, layers)
        else:
            cr.stage1(embed, layers)
            h = cr.stage2(embed, layers)
        got.append([h.clone(), cr.rows.clone()] + [L[c] for L in layers for c in ("k_cache", "v_cache")])
        score = cr.score.clone() if whole else (score, cr.score)
    for a, b in zip(*got):
        assert torch.equal(a, b)
    # fp32: another order of the same sums.  bf16: the queries of the last scoring layer come from
    # a launch of their own, whose tiles may sum in another order; an element on the other side of
    # a tie is a unit (2^-7 of it) away, and a score averages the probabilities of many such rows
    assert torch.allclose(score[0], score[1], rtol=1e-5 if cfg.dtype == "f32" else 2.0 ** -7, atol=0)


@pytest.mark.parametrize("name", sorted(CASES))
def test_chunk_caches_are_those_of_whole_layers(gpu_device, name):
    cfg, inter, embed, layers = setup(name, gpu_device)
    t = 37
    k, v = diagnostics.Diagnostics(cfg, inter, EPS, gpu_device).prefill_cache(embed[:t], layers)
    sub = cfg.with_(n_chunks=1, chunk_len=t - 1, n_query=1)
    cr = model.CarriedRows(sub, inter, EPS, gpu_device, k=t - 1)
    cr.rows[:t - 1] = torch.arange(t - 1, dtype=torch.int32, device=gpu_device)
    full = [dict(L, k_cache=torch.zeros_like(k[0]), v_cache=torch.zeros_like(v[0])) for L in layers]
    cr.stage2(embed[:t].contiguous(), full)
    for li, (L, kk, vv) in enumerate(zip(full, k, v)):
        out = torch.empty_like(kk)
        api.pkv_rope_restore(cr.lc, L["k_cache"], out,
                             -torch.arange(t, dtype=torch.int32, device=gpu_device))
        for a, b in ((out, kk), (L["v_cache"], vv)):
            if li < len(full) - 1:
                assert torch.equal(a, b)
            else:   # a launch without queries: its sums may run in another order (a unit at most)
                a, b = a.float(), b.float()
                assert (a - b).abs().max() <= (1e-5 if cfg.dtype == "f32" else 2.0 ** -7) * b.abs().max()
