"""GPU parity, call by call: every C-ABI entry point against the CPU oracle on
the same seeded inputs.  Sizes span several tiles and a ragged tail; edge
cases (empty, k = 0, k = n, ties, in place, negative and very large positions)
are included.  Tolerances: index work bit-exact; floating point
max|a - b| / max|b| <= 1e-4 (fp32 storage) or 2e-2 (bf16 storage), with tighter
bounds where the arithmetic allows (stated per test)."""

import numpy as np
import pytest
import torch

from oracle import pkv_oracle as O
from paper_2602_02579_amd import api, synth

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def dev(x, dtype, device):
    t = torch.from_numpy(np.ascontiguousarray(x))
    if t.dtype in (torch.float32, torch.float64):
        t = t.to({"f32": torch.float32, "bf16": torch.bfloat16}[dtype])
    return t.to(device)


def host(t):
    return t.detach().to("cpu").to(torch.float64).numpy()


def rel_err(got, want):
    if want.size == 0:
        return 0.0
    return float(np.abs(got - want).max() / max(np.abs(want).max(), 1e-30))


def rnd(seed, shape, dtype, scale=1.0):
    x = np.random.default_rng(seed).standard_normal(shape).astype(np.float32) * np.float32(scale)
    return synth.to_storage(x, dtype)


def lcfg(dtype, hq, hkv, d, hid=256, theta=500000.0):
    return api.LayerCfg(hq, hkv, d, hid, theta, dtype)


# ------------------------------------------------------------------ rope

@pytest.mark.parametrize("dtype,n,hkv,d,theta", [
    ("f32", 1024, 4, 64, 10000.0), ("f32", 333, 2, 32, 10000.0),
    ("bf16", 8192 + 77, 8, 128, 500000.0), ("bf16", 5, 1, 16, 500000.0),
    ("bf16", 1000, 3, 256, 500000.0)])
def test_rope_restore_matches_oracle(gpu_device, dtype, n, hkv, d, theta):
    cfg = lcfg(dtype, hkv, hkv, d, theta=theta)
    x = rnd(1, (n, hkv, d), dtype)
    want = O.rope_restore(x.astype(np.float64), np.arange(n), theta, dtype)
    k_in = dev(x, dtype, gpu_device)
    k_out = torch.empty_like(k_in)
    api.pkv_rope_restore(cfg, k_in, k_out)
    got = host(k_out)
    assert rel_err(got, want) <= TOL[dtype]
    if dtype == "bf16":
        # same bf16 value almost everywhere, never more than one bf16 step off
        diff = np.abs(got - want)
        assert (diff > 0).mean() < 0.02
        assert (diff <= np.abs(want) * 2.0 ** -7 + 1e-6).all()
    else:
        assert np.abs(got - want).max() <= 4e-6


def test_rope_restore_positions_inplace_and_inverse(gpu_device):
    dtype, n, hkv, d, theta = "f32", 700, 2, 64, 500000.0
    cfg = lcfg(dtype, hkv, hkv, d, theta=theta)
    x = rnd(2, (n, hkv, d), dtype)
    pos_np = np.random.default_rng(3).integers(-200000, 200000, size=n).astype(np.int32)
    pos_np[:4] = [0, 131071, -131071, 1]
    want = O.rope_restore(x.astype(np.float64), pos_np, theta, dtype)
    buf = dev(x, dtype, gpu_device)
    pos = torch.from_numpy(pos_np).to(gpu_device)
    api.pkv_rope_restore(cfg, buf, buf, pos)          # in place
    assert np.abs(host(buf) - want).max() <= 4e-6
    assert np.array_equal(host(buf)[0], x[0].astype(np.float64))   # position 0
    api.pkv_rope_restore(cfg, buf, buf, -pos)         # inverse rotation
    assert np.abs(host(buf) - x).max() <= 8e-6
    # pos_base form equals the explicit form
    a = dev(x, dtype, gpu_device)
    b = torch.empty_like(a)
    c = torch.empty_like(a)
    api.pkv_rope_restore(cfg, a, b, None, 32768)
    api.pkv_rope_restore(cfg, a, c, torch.arange(32768, 32768 + n, dtype=torch.int32,
                                                 device=gpu_device))
    assert torch.equal(b, c)


def test_rope_restore_empty_is_a_noop(gpu_device):
    cfg = lcfg("bf16", 8, 8, 128)
    e = torch.empty((0, 8, 128), dtype=torch.bfloat16, device=gpu_device)
    api.pkv_rope_restore(cfg, e, e)


# ------------------------------------------------------------------ scatter

@pytest.mark.parametrize("dtype,hkv,d", [("f32", 4, 64), ("bf16", 8, 128)])
def test_scatter_kv_is_bit_exact(gpu_device, dtype, hkv, d):
    cfg = lcfg(dtype, hkv, hkv, d)
    n_cache, m = 3001, 777
    g = np.random.default_rng(4)
    kc, vc = rnd(5, (n_cache, hkv, d), dtype), rnd(6, (n_cache, hkv, d), dtype)
    kn, vn = rnd(7, (m, hkv, d), dtype), rnd(8, (m, hkv, d), dtype)
    dst = np.sort(g.choice(n_cache, m, replace=False)).astype(np.int32)
    dst[-1] = n_cache - 1
    dst = np.unique(dst).astype(np.int32)
    m = dst.shape[0]
    kn, vn = kn[:m], vn[:m]
    wk, wv = O.scatter_kv(kc, vc, kn, vn, dst)
    tk, tv = dev(kc, dtype, gpu_device), dev(vc, dtype, gpu_device)
    api.pkv_scatter_kv(cfg, dev(kn, dtype, gpu_device), dev(vn, dtype, gpu_device),
                       torch.from_numpy(dst).to(gpu_device), tk, tv)
    assert np.array_equal(host(tk), wk) and np.array_equal(host(tv), wv)
    # gather after scatter returns what was scattered
    assert np.array_equal(host(tk)[dst], kn.astype(np.float64))


# ------------------------------------------------------------------ top-k

def run_topk(score_np, k, device):
    s = torch.from_numpy(score_np.astype(np.float32)).to(device)
    out = torch.full((max(k, 1),), -7, dtype=torch.int32, device=device)
    api.pkv_topk_select(s, k, out)
    return out[:k].cpu().numpy()


@pytest.mark.parametrize("n,k", [(1, 1), (63, 10), (64, 64), (1000, 0), (1000, 1000),
                                 (1024, 204), (32768, 6553), (131072, 26214),
                                 (100003, 99999), (65, 1), (50000, 12345), (65536, 100),
                                 (32769, 32768), (40001, 1), (8192, 1638), (8193, 8000),
                                 (16384, 3277), (12001, 7), (16385, 16000)])
def test_topk_matches_oracle(gpu_device, n, k):
    s = np.random.default_rng(n + k).random(n).astype(np.float32) / n
    assert np.array_equal(run_topk(s, k, gpu_device), O.topk_select(s, k))


def test_topk_score_pointer_not_16_byte_aligned(gpu_device):
    s = np.random.default_rng(77).random(20001).astype(np.float32)
    full = torch.from_numpy(s).to(gpu_device)
    out = torch.empty(5000, dtype=torch.int32, device=gpu_device)
    api.pkv_topk_select(full[1:], 5000, out)      # data pointer offset by 4 bytes
    assert np.array_equal(out.cpu().numpy(), O.topk_select(s[1:], 5000))


def test_topk_ties_negative_values_and_zeros(gpu_device):
    g = np.random.default_rng(9)
    for n, k in [(5000, 1234), (777, 1), (4096, 4095)]:
        s = g.integers(0, 7, size=n).astype(np.float32)          # heavy ties
        assert np.array_equal(run_topk(s, k, gpu_device), O.topk_select(s, k))
    s = np.ones(3000, np.float32)                                 # all equal
    assert np.array_equal(run_topk(s, 700, gpu_device), np.arange(700))
    s = g.standard_normal(2000).astype(np.float32)                # signed
    s[::7] = 0.0
    s[3::7] = -0.0
    assert np.array_equal(run_topk(s, 900, gpu_device), O.topk_select(s, 900))
    assert np.array_equal(run_topk(s, 1500, gpu_device), O.topk_select(s, 1500))


def run_topk_ws(score_t, k, device):
    cfg = lcfg("bf16", 32, 8, 128, 4096)
    n = score_t.shape[0]
    need = api.pkv_workspace_bytes(api.CALL_TOPK_SELECT, cfg, n, 0)
    ws = torch.full((max(need, 256),), 0xAB, dtype=torch.uint8, device=device)   # dirty scratch
    out = torch.full((max(k, 1),), -7, dtype=torch.int32, device=device)
    api.pkv_topk_select(score_t, k, out, ws=ws)
    return out[:k].cpu().numpy(), need


@pytest.mark.parametrize("n,k", [(131072, 26214), (24577, 1), (32768, 6553), (65537, 65537), (100003, 99999),
                                 (262144, 52428), (1 << 20, 1000), (300001, 150000)])
def test_topk_long_vectors_with_a_workspace(gpu_device, n, k):
    """Vectors beyond 65536 scores: the many-workgroup radix select (workspace given)
    against the oracle and against the one-workgroup kernel (no workspace)."""
    g = np.random.default_rng(n ^ k)
    s = (g.random(n).astype(np.float32) ** 4) / n        # skewed, like attention scores
    st = torch.from_numpy(s).to(gpu_device)
    got, need = run_topk_ws(st, k, gpu_device)
    assert need > 0
    want = O.topk_select(s, k)
    assert np.array_equal(got, want)
    assert np.array_equal(run_topk(s, k, gpu_device), want)
    # twice through the same (now used) workspace gives the same indices
    got2, _ = run_topk_ws(st, k, gpu_device)
    assert np.array_equal(got2, want)


def test_topk_long_vectors_ties_signs_and_alignment(gpu_device):
    g = np.random.default_rng(19)
    n = 200001
    s = g.integers(-3, 4, size=n).astype(np.float32)              # heavy ties, both signs
    s[::11] = 0.0
    s[5::11] = -0.0
    st = torch.from_numpy(s).to(gpu_device)
    for k in (1, 77777, 123456, n):
        got, _ = run_topk_ws(st, k, gpu_device)
        assert np.array_equal(got, O.topk_select(s, k))
    got, _ = run_topk_ws(st[1:], 50000, gpu_device)               # pointer offset by 4 bytes
    assert np.array_equal(got, O.topk_select(s[1:], 50000))
    ones = torch.ones(70000, dtype=torch.float32, device=gpu_device)   # all equal
    got, _ = run_topk_ws(ones, 12345, gpu_device)
    assert np.array_equal(got, np.arange(12345))
    cfg = lcfg("bf16", 32, 8, 128, 4096)
    assert api.pkv_workspace_bytes(api.CALL_TOPK_SELECT, cfg, 24576, 0) == 0
    assert api.pkv_workspace_bytes(api.CALL_TOPK_SELECT, cfg, (1 << 22) + 1, 0) == 0


# ------------------------------------------------------------------ score

@pytest.mark.parametrize("dtype,nq,n_ctx,hq,hkv,d", [
    ("f32", 16, 1024, 4, 4, 64), ("f32", 3, 301, 4, 2, 32),
    ("bf16", 64, 2048 + 37, 32, 8, 128), ("bf16", 5, 100, 8, 8, 64),
    ("bf16", 7, 515, 10, 2, 128)])
def test_query_score_matches_oracle(gpu_device, dtype, nq, n_ctx, hq, hkv, d):
    cfg = lcfg(dtype, hq, hkv, d)
    q = rnd(10, (nq, hq, d), dtype, 1.3)
    k = rnd(11, (n_ctx, hkv, d), dtype)
    want = O.query_score(q.astype(np.float64), k.astype(np.float64))
    score = torch.full((n_ctx,), 9.0, dtype=torch.float32, device=gpu_device)
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, cfg, n_ctx, nq), 256),
                     dtype=torch.uint8, device=gpu_device)
    tq, tk = dev(q, dtype, gpu_device), dev(k, dtype, gpu_device)
    api.pkv_query_score(cfg, tq, tk, score, accumulate=False, ws=ws)
    got = host(score)
    # fp32 arithmetic on identical stored inputs: far inside the paper-level bar
    assert rel_err(got, want) <= 1e-4
    assert abs(got.sum() - 1.0) < 1e-4
    # layer fusion: adding the same layer again doubles the score
    api.pkv_query_score(cfg, tq, tk, score, accumulate=True, ws=ws)
    want2 = O.fuse_score(O.fuse_score(np.zeros(n_ctx), want), want)
    assert rel_err(host(score), want2) <= 1e-4
    # deterministic
    s2 = torch.empty_like(score)
    s3 = torch.empty_like(score)
    api.pkv_query_score(cfg, tq, tk, s2, ws=ws)
    api.pkv_query_score(cfg, tq, tk, s3, ws=ws)
    assert torch.equal(s2, s3)


def test_query_score_late_keys_far_above_the_first_tile(gpu_device):
    """Scores that grow by hundreds of nats after the first 64 keys of a split: the
    head_dim-128 kernel fixes its softmax reference on the first tile and must raise it
    (rescaling its sums) when later probabilities leave the safe range."""
    dtype, nq, n_ctx, hq, hkv, d = "bf16", 40, 3000, 8, 2, 128
    cfg = lcfg(dtype, hq, hkv, d)
    q = rnd(40, (nq, hq, d), dtype, 1.0)
    k = rnd(41, (n_ctx, hkv, d), dtype, 0.05)
    q[10:, 2, :] = 4.0                       # some columns only
    k[200::5, 0, :] = 4.0                    # aligned keys: q.k ~ 2048 -> ~180 nats
    k[1500::11, 0, :] = 6.0                  # and another step up later on
    q, k = synth.to_storage(q, dtype), synth.to_storage(k, dtype)
    want = O.query_score(q.astype(np.float64), k.astype(np.float64))
    score = torch.empty(n_ctx, dtype=torch.float32, device=gpu_device)
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, cfg, n_ctx, nq), 256),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_query_score(cfg, dev(q, dtype, gpu_device), dev(k, dtype, gpu_device), score,
                        accumulate=False, ws=ws)
    got = host(score)
    assert np.isfinite(got).all()
    assert rel_err(got, want) <= 1e-4
    assert abs(got.sum() - 1.0) < 1e-4


def test_query_score_custom_scale(gpu_device):
    cfg = lcfg("f32", 2, 2, 32)
    q, k = rnd(12, (4, 2, 32), "f32"), rnd(13, (200, 2, 32), "f32")
    want = O.query_score(q.astype(np.float64), k.astype(np.float64), scale=0.05)
    score = torch.empty(200, dtype=torch.float32, device=gpu_device)
    ws = torch.empty(4096, dtype=torch.uint8, device=gpu_device)
    api.pkv_query_score(cfg, dev(q, "f32", gpu_device), dev(k, "f32", gpu_device), score,
                        softmax_scale=0.05, ws=ws)
    assert rel_err(host(score), want) <= 1e-4


# ------------------------------------------------------------------ projection

@pytest.mark.parametrize("dtype,m,hq,hkv,d,hid,theta", [
    ("f32", 220, 4, 4, 64, 256, 10000.0), ("f32", 37, 4, 2, 32, 64, 10000.0),
    ("bf16", 300, 32, 8, 128, 1024, 500000.0), ("bf16", 65, 4, 4, 64, 128, 500000.0),
    ("bf16", 129, 10, 2, 128, 512, 500000.0), ("bf16", 257, 4, 2, 128, 160, 500000.0),
    ("bf16", 1, 2, 2, 128, 4096, 500000.0)])
def test_gather_qkv_proj_matches_oracle(gpu_device, dtype, m, hq, hkv, d, hid, theta):
    cfg = lcfg(dtype, hq, hkv, d, hid, theta)
    n_rows = 2 * m + 11
    g = np.random.default_rng(14)
    hidden = rnd(15, (n_rows, hid), dtype)
    wq = rnd(16, (hq * d, hid), dtype, 1.0 / np.sqrt(hid))
    wk = rnd(17, (hkv * d, hid), dtype, 1.0 / np.sqrt(hid))
    wv = rnd(18, (hkv * d, hid), dtype, 1.0 / np.sqrt(hid))
    rows = np.sort(g.choice(n_rows, m, replace=False)).astype(np.int32)
    pos = (rows.astype(np.int64) * 57 + 3).astype(np.int32)       # positions != rows
    wantq, wantk, wantv = O.project_qkv_rows(
        hidden.astype(np.float64), rows, pos, wq.astype(np.float64),
        wk.astype(np.float64), wv.astype(np.float64), hq, hkv, d, theta, dtype)
    dt = cfg.torch_dtype
    qo = torch.empty((m, hq, d), dtype=dt, device=gpu_device)
    ko = torch.empty((m, hkv, d), dtype=dt, device=gpu_device)
    vo = torch.empty((m, hkv, d), dtype=dt, device=gpu_device)
    args = (dev(hidden, dtype, gpu_device), torch.from_numpy(rows).to(gpu_device),
            torch.from_numpy(pos).to(gpu_device), dev(wq, dtype, gpu_device),
            dev(wk, dtype, gpu_device), dev(wv, dtype, gpu_device))
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_GATHER_QKV_PROJ, cfg, 0, m), 256),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_gather_qkv_proj(cfg, *args, qo, ko, vo, ws=ws)
    for got, want in ((qo, wantq), (ko, wantk), (vo, wantv)):
        assert rel_err(host(got), want) <= TOL[dtype]
    # Q only / KV only variants write the same bits
    q2 = torch.empty_like(qo)
    api.pkv_gather_qkv_proj(cfg, args[0], args[1], args[2], args[3], None, None,
                            q2, None, None, ws=ws)
    assert torch.equal(q2, qo)
    k2, v2 = torch.empty_like(ko), torch.empty_like(vo)
    api.pkv_gather_qkv_proj(cfg, args[0], args[1], args[2], None, args[4], args[5],
                            None, k2, v2, ws=ws)
    assert torch.equal(k2, ko) and torch.equal(v2, vo)
    # identity gather
    q3 = torch.empty_like(qo)
    api.pkv_gather_qkv_proj(cfg, args[0][rows.astype(np.int64)].contiguous(), None,
                            args[2], args[3], None, None, q3, None, None, ws=ws)
    assert torch.equal(q3, qo)


@pytest.mark.parametrize("hid", [1024, 1152])
def test_gather_qkv_proj_more_tiles_than_cus(gpu_device, hid):
    """2900 rows x (32 + 2 x 8) heads = 288 tiles of 256 x 256: more than one round of the 256
    CUs, a ragged last token tile, and the XCD-aware tile order over more than one group."""
    dtype, m, hq, hkv, d = "bf16", 2900, 32, 8, 128
    cfg = lcfg(dtype, hq, hkv, d, hid)
    g = np.random.default_rng(91)
    n_rows = 3100
    hidden = rnd(92, (n_rows, hid), dtype)
    w = [rnd(93 + i, (h * d, hid), dtype, 1.0 / np.sqrt(hid)) for i, h in enumerate((hq, hkv, hkv))]
    rows = np.sort(g.choice(n_rows, m, replace=False)).astype(np.int32)
    pos = np.sort(g.choice(200000, m, replace=False)).astype(np.int32)
    want = O.project_qkv_rows(hidden.astype(np.float64), rows, pos,
                              *[x.astype(np.float64) for x in w], hq, hkv, d, cfg.rope_theta,
                              dtype)
    args = (dev(hidden, dtype, gpu_device), torch.from_numpy(rows).to(gpu_device),
            torch.from_numpy(pos).to(gpu_device), *[dev(x, dtype, gpu_device) for x in w])
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_GATHER_QKV_PROJ, cfg, 0, m), 256),
                     dtype=torch.uint8, device=gpu_device)
    outs = [torch.full((m, h, d), float("nan"), dtype=cfg.torch_dtype, device=gpu_device)
            for h in (hq, hkv, hkv)]
    api.pkv_gather_qkv_proj(cfg, *args, *outs, ws=ws)
    for o, wnt in zip(outs, want):
        assert torch.isfinite(o.float()).all()
        assert rel_err(host(o), wnt) <= TOL[dtype]


# ------------------------------------------------------------------ attention

@pytest.mark.parametrize("dtype,m,n_keys,hq,hkv,d", [
    ("f32", 220, 1040, 4, 4, 64), ("f32", 19, 130, 4, 2, 32),
    ("bf16", 333, 2048 + 61, 32, 8, 128), ("bf16", 70, 300, 4, 4, 64),
    ("bf16", 100, 777, 10, 2, 128), ("bf16", 1, 1, 32, 8, 128),
    ("bf16", 300, 500, 4, 1, 128), ("bf16", 150, 321, 6, 3, 128), ("bf16", 90, 200, 48, 3, 128)])
def test_sparse_row_attn_matches_oracle(gpu_device, dtype, m, n_keys, hq, hkv, d, v_source):
    cfg = lcfg(dtype, hq, hkv, d)
    g = np.random.default_rng(19)
    q = rnd(20, (m, hq, d), dtype, 1.2)
    kc, vc = rnd(21, (n_keys, hkv, d), dtype), rnd(22, (n_keys, hkv, d), dtype)
    pos = np.sort(g.choice(n_keys, m, replace=n_keys < m)).astype(np.int32)
    pos[0] = 0
    pos[-1] = n_keys - 1
    want, want_lse = O.sparse_row_attn(q.astype(np.float64), kc.astype(np.float64),
                                       vc.astype(np.float64), pos, dtype=dtype)
    dt = cfg.torch_dtype
    out = torch.empty((m, hq, d), dtype=dt, device=gpu_device)
    lse = torch.empty((m, hq), dtype=torch.float32, device=gpu_device)
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m), 256),
                     dtype=torch.uint8, device=gpu_device)
    args = (dev(q, dtype, gpu_device), dev(kc, dtype, gpu_device), dev(vc, dtype, gpu_device))
    api.pkv_sparse_row_attn(cfg, *args, torch.from_numpy(pos).to(gpu_device), out, lse, ws=ws)
    assert rel_err(host(out), want) <= TOL[dtype]
    # bf16: the normaliser sums bf16-rounded probabilities (2^-9 relative each)
    assert np.abs(host(lse) - want_lse).max() <= (4e-3 if dtype == "bf16" else 1e-3)
    # row order does not matter: a shuffled row set gives the same rows
    perm = g.permutation(m)
    out2 = torch.empty_like(out)
    api.pkv_sparse_row_attn(cfg, args[0][perm].contiguous(), args[1], args[2],
                            torch.from_numpy(pos[perm]).to(gpu_device), out2, None, ws=ws)
    assert rel_err(host(out2), want[perm]) <= TOL[dtype]


@pytest.mark.parametrize("hq,hkv,m,n_keys", [(16, 16, 4400, 600), (32, 8, 2200, 900)])
def test_sparse_row_attn_more_row_tiles_than_workgroups(gpu_device, hq, hkv, m, n_keys, v_source):
    """More (kv head, row tile) pairs than the launch has workgroups, so that every
    workgroup claims several and the heads run out at different times; rows in no
    particular order, so that the tiles differ in cost.  Who claims a tile must not
    matter: a second call gives the same bits."""
    dtype, d = "bf16", 128
    cfg = lcfg(dtype, hq, hkv, d)
    g = np.random.default_rng(41)
    q = rnd(42, (m, hq, d), dtype, 1.2)
    kc, vc = rnd(43, (n_keys, hkv, d), dtype), rnd(44, (n_keys, hkv, d), dtype)
    pos = g.integers(0, n_keys, m).astype(np.int32)
    pos[:300] = np.sort(pos[:300])          # a few cheap tiles among the expensive ones
    pos[:300] //= 8
    pos[-1] = n_keys - 1
    n_tiles = -(-m // (256 // (hq // hkv)))
    props = torch.cuda.get_device_properties(gpu_device)
    assert n_tiles * hkv > props.multi_processor_count
    want, want_lse = O.sparse_row_attn(q.astype(np.float64), kc.astype(np.float64),
                                       vc.astype(np.float64), pos, dtype=dtype)
    out = torch.empty((m, hq, d), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.empty((m, hq), dtype=torch.float32, device=gpu_device)
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m), 256),
                     dtype=torch.uint8, device=gpu_device)
    args = (dev(q, dtype, gpu_device), dev(kc, dtype, gpu_device), dev(vc, dtype, gpu_device),
            torch.from_numpy(pos).to(gpu_device))
    api.pkv_sparse_row_attn(cfg, *args, out, lse, ws=ws)
    assert rel_err(host(out), want) <= TOL[dtype]
    assert np.abs(host(lse) - want_lse).max() <= 4e-3
    out2, lse2 = torch.empty_like(out), torch.empty_like(lse)
    ws.fill_(0xff)                           # the call must not rely on what the last one left
    api.pkv_sparse_row_attn(cfg, *args, out2, lse2, ws=ws)
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("hq,hkv,m,n_keys,query_rows", [
    (32, 8, 128, 8192 + 128, True),      # Stage I: the query rows alone, 16 (head, tile) pairs
    (32, 8, 200, 8300, False),           # rows anywhere: some see only the first key range
    (8, 2, 500, 5000, False), (40, 8, 70, 6666, False)])
def test_sparse_row_attn_few_rows_split_over_keys(gpu_device, hq, hkv, m, n_keys, query_rows, v_source):
    """Fewer (kv head, row tile) pairs than CUs: the keys of a tile are cut into ranges
    that run as separate jobs and are merged (rows that end inside a range, rows that
    never reach a range, a ragged last range)."""
    dtype, d = "bf16", 128
    cfg = lcfg(dtype, hq, hkv, d)
    g = np.random.default_rng(51)
    q = rnd(52, (m, hq, d), dtype, 1.2)
    kc, vc = rnd(53, (n_keys, hkv, d), dtype), rnd(54, (n_keys, hkv, d), dtype)
    if query_rows:
        pos = np.arange(n_keys - m, n_keys, dtype=np.int32)
    else:
        pos = np.sort(g.integers(0, n_keys, m)).astype(np.int32)
        pos[0], pos[1], pos[-1] = 0, 1023, n_keys - 1
    want, want_lse = O.sparse_row_attn(q.astype(np.float64), kc.astype(np.float64),
                                       vc.astype(np.float64), pos, dtype=dtype)
    out = torch.empty((m, hq, d), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.empty((m, hq), dtype=torch.float32, device=gpu_device)
    need = api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m)
    # the launcher did plan ranges: the scratch holds fp32 partial results for two or more
    assert need > hkv * d * (n_keys + 64) * 2 + 1.5 * m * hq * (d + 1) * 4
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device=gpu_device)
    ws.fill_(0xff)
    args = (dev(q, dtype, gpu_device), dev(kc, dtype, gpu_device), dev(vc, dtype, gpu_device),
            torch.from_numpy(pos).to(gpu_device))
    api.pkv_sparse_row_attn(cfg, *args, out, lse, ws=ws)
    assert rel_err(host(out), want) <= TOL[dtype]
    assert np.abs(host(lse) - want_lse).max() <= 4e-3
    out2 = torch.empty_like(out)
    api.pkv_sparse_row_attn(cfg, *args, out2, None, ws=ws)
    assert torch.equal(out, out2)


@pytest.mark.parametrize("seed", range(12))
def test_sparse_row_attn_random_shapes(gpu_device, seed, v_source):
    """Seeded random geometry, row count, cache length and row limits (head_dim 128,
    bf16): whatever tiling, key ranges and claim order the launcher picks, the rows match."""
    g = np.random.default_rng(1000 + seed)
    hq, hkv = [(32, 8), (8, 8), (16, 2), (12, 4), (40, 8), (4, 1), (64, 8)][seed % 7]
    m = int(g.integers(1, 900))
    n_keys = int(g.integers(1, 9000))
    dtype, d = "bf16", 128
    cfg = lcfg(dtype, hq, hkv, d)
    q = rnd(2000 + seed, (m, hq, d), dtype, 1.1)
    kc, vc = rnd(3000 + seed, (n_keys, hkv, d), dtype), rnd(4000 + seed, (n_keys, hkv, d), dtype)
    pos = g.integers(0, n_keys, m).astype(np.int32)
    if seed % 3 == 0:
        pos = np.sort(pos)
    if seed % 4 == 1:
        pos[:] = n_keys - 1                      # every row sees the whole cache
    want, want_lse = O.sparse_row_attn(q.astype(np.float64), kc.astype(np.float64),
                                       vc.astype(np.float64), pos, dtype=dtype)
    out = torch.empty((m, hq, d), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.empty((m, hq), dtype=torch.float32, device=gpu_device)
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m), 256),
                     dtype=torch.uint8, device=gpu_device)
    ws.fill_(0x5a)
    api.pkv_sparse_row_attn(cfg, dev(q, dtype, gpu_device), dev(kc, dtype, gpu_device),
                            dev(vc, dtype, gpu_device), torch.from_numpy(pos).to(gpu_device),
                            out, lse, ws=ws)
    assert rel_err(host(out), want) <= TOL[dtype], (hq, hkv, m, n_keys)
    assert np.abs(host(lse) - want_lse).max() <= 4e-3, (hq, hkv, m, n_keys)


def test_sparse_row_attn_closed_forms(gpu_device):
    dtype, hq, hkv, d, n_keys = "bf16", 8, 2, 128, 500
    cfg = lcfg(dtype, hq, hkv, d)
    q = rnd(23, (3, hq, d), dtype)
    kc = rnd(24, (n_keys, hkv, d), dtype)
    vc = np.broadcast_to(rnd(25, (1, hkv, d), dtype), (n_keys, hkv, d)).copy()
    out = torch.empty((3, hq, d), dtype=torch.bfloat16, device=gpu_device)
    pos = torch.tensor([0, 250, 499], dtype=torch.int32, device=gpu_device)
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, 3), 256),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_sparse_row_attn(cfg, dev(q, dtype, gpu_device), dev(kc, dtype, gpu_device),
                            dev(vc, dtype, gpu_device), pos, out, None, ws=ws)
    got = host(out)
    for h in range(hq):   # constant values come back (up to bf16 rounding of the mean)
        assert np.abs(got[:, h] - vc[0, h // 4]).max() <= 2e-2 * np.abs(vc[0]).max()


# 700 keys: the running maximum of the short-cache kernel with the values as the cache holds
# them, the pipelined kernel on the transposed copy; 4500: the keys of a tile run as 18 ranges
@pytest.mark.parametrize("n_keys", [700, 4500])
def test_sparse_row_attn_scores_far_above_the_first_keys(gpu_device, n_keys, v_source):
    """Late keys whose scores exceed everything among a row's first 32 keys by
    hundreds of nats: the fixed-reference first attempt of the pipelined head_dim-128
    kernels cannot represent them, and the workgroup must do its job again."""
    dtype, hq, hkv, d, m = "bf16", 8, 2, 128, 150
    cfg = lcfg(dtype, hq, hkv, d)
    g = np.random.default_rng(31)
    q = rnd(32, (m, hq, d), dtype, 1.0)
    kc, vc = rnd(33, (n_keys, hkv, d), dtype, 0.05), rnd(34, (n_keys, hkv, d), dtype)
    # from key 300 on, keys of kv head 0 are aligned with the queries of rows 60..149
    # of q head 1 (dot product ~ 128 * 16 -> ~180 nats after the 1/sqrt(d) scale);
    # kv head 1 and the other rows stay ordinary
    q[60:, 1, :] = 4.0
    kc[300::7, 0, :] = 4.0
    q, kc = synth.to_storage(q, dtype), synth.to_storage(kc, dtype)
    pos = np.sort(g.choice(n_keys, m, replace=False)).astype(np.int32)
    pos[-1] = n_keys - 1
    want, want_lse = O.sparse_row_attn(q.astype(np.float64), kc.astype(np.float64),
                                       vc.astype(np.float64), pos, dtype=dtype)
    out = torch.empty((m, hq, d), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.empty((m, hq), dtype=torch.float32, device=gpu_device)
    ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, cfg, n_keys, m), 256),
                     dtype=torch.uint8, device=gpu_device)
    api.pkv_sparse_row_attn(cfg, dev(q, dtype, gpu_device), dev(kc, dtype, gpu_device),
                            dev(vc, dtype, gpu_device), torch.from_numpy(pos).to(gpu_device),
                            out, lse, ws=ws)
    got, got_lse = host(out), host(lse)
    assert np.isfinite(got).all() and np.isfinite(got_lse).all()
    assert rel_err(got, want) <= TOL[dtype]
    assert np.abs(got_lse - want_lse).max() <= 4e-3 * max(1.0, np.abs(want_lse).max() / 10)


# ------------------------------------------------------------------ errors

def test_host_checked_errors(gpu_device):
    cfg = lcfg("bf16", 32, 8, 128, 4096)
    k = torch.zeros((4, 8, 128), dtype=torch.bfloat16, device=gpu_device)
    bad = api.LayerCfg(32, 5, 128, 4096, 5e5, "bf16")
    with pytest.raises(api.PkvError) as e:
        api.pkv_rope_restore(bad, k[:, :5].contiguous(), k[:, :5].contiguous())
    assert e.value.status == 2
    odd = api.LayerCfg(8, 8, 72, 4096, 5e5, "bf16")
    x = torch.zeros((4, 8, 72), dtype=torch.bfloat16, device=gpu_device)
    with pytest.raises(api.PkvError) as e:
        api.pkv_rope_restore(odd, x, x)
    assert e.value.status == 3
    s = torch.zeros(10, dtype=torch.float32, device=gpu_device)
    o = torch.zeros(20, dtype=torch.int32, device=gpu_device)
    with pytest.raises(api.PkvError) as e:
        api.pkv_topk_select(s, 11, o)
    assert e.value.status == 2
    q = torch.zeros((2, 32, 128), dtype=torch.bfloat16, device=gpu_device)
    with pytest.raises(api.PkvError) as e:
        api.pkv_query_score(cfg, q, k, s[:4].contiguous(), ws=None)
    assert e.value.status == 4
