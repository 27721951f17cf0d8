"""A whole decoder layer in one call: what its host checks refuse, and (on the GPU) the same bits as
the calls it stands for (fp32: the same values to rounding), in every form: with and without block
variants, both ways of scoring, chunks, and the three places where it may stop."""

import ctypes
import os

import pytest
import torch

from paper_2602_02579_amd import api

EPS = 1e-5


def test_bad_calls_are_refused_without_a_gpu():
    if not os.path.exists(api.library_path()):
        pytest.skip("libpkv.so not built")
    lib = api.load_library()
    cfg = api.LayerCfg(8, 2, 128, 256, 1e4, "bf16")

    def status(**fields):
        c = api.LayerCall(eps=EPS, inter=256, **fields)
        return lib.pkv_layer_rows(cfg._ref, ctypes.byref(c), None)
    assert lib.pkv_layer_rows(cfg._ref, None, None) == 1
    assert lib.pkv_layer_rows(None, ctypes.byref(api.LayerCall()), None) == 1
    assert status(stop=3) == 2 and status(stop=-1) == 2 and status(chunk_len=-1) == 2
    assert status(m=4, n_cache=5, chunk_len=2) == 2        # chunks are all of the caches
    assert status(m=4, n_cache=4, chunk_len=2, score=64) == 2
    assert status(m=-1, n_cache=4) == 2
    assert status(m=4, n_cache=8) == 1                     # null buffers
    assert status(m=0, n_cache=4) == 0


def test_shapes_are_checked_before_anything_is_enqueued():
    cfg = api.LayerCfg(8, 2, 128, 256, 1e4, "bf16")
    new = lambda *s: torch.zeros(s, dtype=torch.bfloat16)   # noqa: E731
    with pytest.raises(ValueError, match="h must be"):
        api.pkv_layer_rows(cfg, new(3, 256), new(4, 256), new(4, 8, 128), new(4, 8, 128),
                           new(4, 64), 4, {}, (), new(4, 2, 128), new(4, 2, 128),
                           torch.zeros(4), torch.zeros(4), EPS, new(1))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,variant", [("f32", ""), ("bf16", ""), ("bf16", "bias"),
                                           ("bf16", "norm")])
@pytest.mark.parametrize("form", ["plain", "score", "fused", "scores_only", "chunks", "caches"])
def test_same_bits_as_the_calls(gpu_device, dtype, variant, form):
    hq, hkv, d, hid, inter, n_ctx = (4, 4, 64, 64, 96, 128) if dtype == "f32" else \
        (8, 2, 128, 256, 512, 128)
    m = 21
    cfg = api.LayerCfg(hq, hkv, d, hid, 1e4, dtype)
    dt = cfg.torch_dtype
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(5)

    def mat(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=gpu_device) * scale).to(dt)
    chunked = form in ("chunks", "caches")
    n_cache = m if chunked else n_ctx + m
    L = dict(w_in=mat(hid), w_post=mat(hid), wq=mat(hq * d, hid, scale=.1),
             wk=mat(hkv * d, hid, scale=.1), wv=mat(hkv * d, hid, scale=.1),
             wo=mat(hid, hq * d, scale=.1), w_gate=mat(inter, hid, scale=.1),
             w_up=mat(inter, hid, scale=.1), w_down=mat(hid, inter, scale=.1))
    if variant == "bias":
        L.update(bq=mat(hq * d), bk=mat(hkv * d), bv=mat(hkv * d))
    elif variant == "norm":
        L.update(q_norm=mat(d), k_norm=mat(d))
    var = {v: L[v] for v in ("bq", "bk", "bv", "q_norm", "k_norm") if v in L}
    rows = torch.arange(n_cache - m, n_cache, dtype=torch.int32, device=gpu_device)
    pos = rows % 8 if chunked else rows
    h0, k0, v0 = mat(m, hid), mat(n_cache, hkv, d), mat(n_cache, hkv, d)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device=gpu_device)
    if form == "fused" and dtype == "f32":
        pytest.skip("the fused first stage is bf16")

    def buffers():
        new = lambda *s: torch.zeros((m + 2,) + s, dtype=dt, device=gpu_device)   # noqa: E731
        h = new(hid)
        h[:m] = h0
        return dict(h=h, x=new(hid), q=new(hq, d), attn=new(hq, d), g=new(inter),
                    k=k0.clone(), v=v0.clone(),
                    score=torch.ones(n_ctx, device=gpu_device),
                    lse=torch.zeros((m, hq), device=gpu_device))
    a, b = buffers(), buffers()
    scoring = form in ("score", "fused", "scores_only")
    api.pkv_layer_rows(
        cfg, a["h"], a["x"], a["q"], a["attn"], a["g"], m, L, tuple(var), a["k"], a["v"], pos,
        rows, EPS, ws, score=a["score"] if scoring else None,
        lse_ctx=a["lse"] if form == "fused" else None, n_ctx=n_ctx, accumulate=True,
        chunk_len=8 if chunked else 0,
        stop={"caches": api.LAYER_TO_CACHES, "scores_only": api.LAYER_TO_SCORES}.get(form, 0))

    h, x, q, attn, g = (b[name][:m] for name in ("h", "x", "q", "attn", "g"))
    api.pkv_rmsnorm_rows(h, None, L["w_in"], EPS, x)
    api.pkv_gather_qkv_proj_scatter(cfg, x, None, pos, L["wq"], L["wk"], L["wv"],
                                    None if form == "caches" else q, b["k"], b["v"], rows, ws=ws,
                                    norm_eps=EPS, **var)
    if form == "chunks":
        api.pkv_chunk_attn(cfg, q, b["k"], b["v"], pos, attn, 8, ws=ws)
    elif form == "fused":
        api.pkv_sparse_row_attn_ctx_lse(cfg, q, b["k"], b["v"], rows, attn, None, b["lse"], n_ctx,
                                        ws=ws)
        api.pkv_query_score_lse(cfg, q, b["k"][:n_ctx], b["lse"], None, b["score"],
                                accumulate=True, ws=ws)
    elif form != "caches":
        if scoring:
            api.pkv_query_score(cfg, q, b["k"][:n_ctx], b["score"], accumulate=True, ws=ws)
        api.pkv_sparse_row_attn(cfg, q, b["k"], b["v"], rows, attn, None, ws=ws)
    if form not in ("caches", "scores_only"):
        api.pkv_linear_rows(attn.view(m, -1), L["wo"], h, h, ws=ws)
        api.pkv_rmsnorm_rows(h, None, L["w_post"], EPS, x)
        api.pkv_swiglu_rows(x, L["w_gate"], L["w_up"], g, ws=ws)
        api.pkv_linear_rows(g, L["w_down"], h, h, ws=ws)
    for name in a:
        if dtype == "bf16":
            assert torch.equal(a[name], b[name]), name
        elif name != "x":      # x is not written where a launch normalises the rows itself
            # fp32, the normalisations' sums in another order and, in the gated layer of so few rows,
            # another kernel's.  One stage: a sum of 64 products of rows that are off by the
            # order of 64 squares, (64 + 32) units of 2^-24 at most; scores, attention and what
            # follows have three more sums of at most 150 terms behind it.
            tol = 96 * 2.0 ** -24 if name in ("q", "k", "v") else 2e-5
            assert (a[name] - b[name]).abs().max() <= tol * max(1.0, b[name].abs().max()), name


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d,hid,m", [(8, 8, 128, 1024, 500), (2, 2, 128, 5120, 2100),
                                            (2, 2, 128, 256, 1), (4, 4, 64, 256, 33)])
def test_angles_out_of_the_norms_launch(gpu_device, hq, hkv, d, hid, m):
    """A workgroup per row, a wave per row in registers and not, and the 256 x 128 kernel: Q, K and V
    are those of the two calls, which make the table in a launch of its own."""
    cfg = api.LayerCfg(hq, hkv, d, hid, 1e4, "bf16")
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(m)

    def mat(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=gpu_device) * scale).to(torch.bfloat16)
    L = dict(w_in=mat(hid), w_post=mat(hid), wq=mat(hq * d, hid, scale=.05),
             wk=mat(hkv * d, hid, scale=.05), wv=mat(hkv * d, hid, scale=.05),
             wo=mat(hid, hq * d), w_gate=mat(64, hid), w_up=mat(64, hid), w_down=mat(hid, 64))
    h = mat(m, hid)
    pos = torch.randperm(3 * m, generator=gen, device=gpu_device)[:m].to(torch.int32)
    rows = torch.randperm(m, generator=gen, device=gpu_device).to(torch.int32)
    ws = torch.empty(256 << 20, dtype=torch.uint8, device=gpu_device)
    new = lambda *s: torch.zeros((m,) + s, dtype=torch.bfloat16, device=gpu_device)   # noqa: E731
    out = [(new(hid), new(hq, d), new(hkv, d), new(hkv, d)) for _ in range(2)]
    x, q, k, v = out[0]
    api.pkv_layer_rows(cfg, h, x, q, new(hq, d), new(64), m, L, (), k, v, pos, rows, EPS, ws,
                       score=torch.zeros(m, device=gpu_device), n_ctx=m,
                       stop=api.LAYER_TO_SCORES)
    x, q, k, v = out[1]
    api.pkv_rmsnorm_rows(h, None, L["w_in"], EPS, x)
    ws.fill_(255)
    api.pkv_gather_qkv_proj_scatter(cfg, x, None, pos, L["wq"], L["wk"], L["wv"], q, k, v, rows,
                                    ws=ws)
    for a, b in zip(*out):
        assert torch.equal(a, b)
