"""Benchmark of the ProphetKV selective-recompute hot path on one MI355X.

A step is one pass of the whole hot path over one synthetic layer of the 32k
configuration (Llama-3-8B geometry, 64 x 512-token chunks, 128 query tokens,
r = 0.2): restore RoPE, project the query rows, score, select, project the
selected + query rows, scatter, attend.  Inputs are resident in HBM before the
timed region.  Prints ONE JSON line.

After the timed steps (and outside `value`) it also times the same configuration as
a small stacked model with the hidden states carried through the layers - Stage I on
the query rows, Stage II on the selected + query rows, each layer with its output
projection and gated MLP (Llama-3-8B widths) - and reports it as `carried_model`.

Also outside `value`: `extras` (the same pass at ratios 0.1 / 0.4, at 8k and 128k
context and through a 32-layer stack with scoring fused over 2 layers, all on device-side
random draws), `bandwidth` (the HBM-bound calls cold - rotating over more than 512 MB of
buffers so that the 256 MB Infinity Cache cannot serve them - and warm, next to a plain
copy measured the same way) and `diagnostics` (selection overlap ratios of Sec. 3.1 on a
small random model, planted-token hit rates of two criteria at the benchmark shape).

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config 3]
                    [--no-cpu-baseline] [--model-layers L] [--no-extras]
"""

from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np
import torch

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

from paper_2602_02579_amd import api, model, pipeline, synth  # noqa: E402

PEAK_BF16_TFLOPS = 2500.0    # MI355X dense bf16 MFMA
# HBM bytes per pkv_sparse_row_attn call (its main kernel 1.897e9, the V^T copy before it 0.135e9),
# from the FETCH_SIZE / WRITE_SIZE counter runs summarised in profiles/hot_path_cfg3_hbm_traffic.txt
# (counters cannot be read from inside this process; the figure is for that workload only)
MEASURED_ATTN_TRAFFIC_BYTES = {"cfg3-llama8b-32k": 2.031e9}
TRAFFIC_SOURCE = ("profiles/hot_path_cfg3_hbm_traffic.txt (rocprofv3 --pmc FETCH_SIZE / "
                  "WRITE_SIZE runs of this program, commands in the file; not read live)")
PEAK_F32_TFLOPS = 157.3
PEAK_HBM_GBS = 8000.0


# --------------------------------------------------------------------------
# workload on the GPU: seeded draws, planted with the library's own calls
# --------------------------------------------------------------------------

def gpu_callables(cfg, layer, device):
    """Rotated-query block and rotation for the planting step, computed with
    the HIP library (the generator itself holds no method arithmetic)."""
    lc = pipeline.layer_cfg(cfg)
    dt = lc.torch_dtype
    hidden = torch.from_numpy(layer["hidden"]).to(dt).to(device)
    wq = torch.from_numpy(layer["wq"]).to(dt).to(device)

    def project_q(rows):
        r = torch.from_numpy(np.asarray(rows, dtype=np.int32)).to(device)
        q = torch.empty((len(rows), cfg.n_q_heads, cfg.head_dim), dtype=dt, device=device)
        ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_GATHER_QKV_PROJ, lc, 0, len(rows)),
                             256), dtype=torch.uint8, device=device)
        api.pkv_gather_qkv_proj(lc, hidden, r, r, wq, None, None, q, None, None, ws=ws)
        return q.float().cpu().numpy()

    f32 = api.LayerCfg(cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.hidden,
                       cfg.theta, "f32")

    def rotate(x, pos):
        t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(device)
        p = torch.from_numpy(np.asarray(pos, dtype=np.int32)).to(device)
        o = torch.empty_like(t)
        api.pkv_rope_restore(f32, t, o, p)
        return o.cpu().numpy()
    return project_q, rotate


def build_gpu_workload(cfg, device):
    """The seeded host draws with plants for the scoring layers; the layers behind them
    (config 4 has 30 more) only feed Stage II and are drawn on the device, same
    distributions, to keep the set-up short.  Returns the layers and the plant index sets
    of the first layer."""
    layers, plants = [], None
    for li in range(cfg.n_layers):
        if li >= cfg.n_score_layers:
            layers.extend(random_layers(cfg, device, cfg.n_layers - li, seed=100 + cfg.seed))
            break
        layer = synth.make_layer(cfg, li)
        pq, rot = gpu_callables(cfg, layer, device)
        info = synth.plant(cfg, layer, li, pq, rot)
        if li == 0:
            plants = dict(relevant=info["relevant"], salient=info["salient"])
        layers.append(pipeline.upload_layer(cfg, layer, device))
        del layer
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return layers, plants


def random_layers(cfg, device, n_layers, seed):
    """Hot-path layers drawn on the device (the distributions of synth.make_layer, nothing
    planted): for the workloads outside `value`, where only the shapes matter."""
    dt = pipeline.layer_cfg(cfg).torch_dtype
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    n, qn = cfg.n_ctx, cfg.n_query
    hq, hkv, d, hid = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.hidden

    def normal(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=device) * scale).to(dt)

    out = []
    for _ in range(n_layers):
        hidden = torch.randn((n + qn, hid), generator=gen, device=device)
        hidden[:n] += 0.5 * torch.randn(hid, generator=gen, device=device)
        hidden[n:] = torch.randn(hid, generator=gen, device=device) + 0.3 * hidden[n:]
        L = dict(k_nope=normal(n, hkv, d), hidden=hidden.to(dt),
                 wq=normal(hq * d, hid, scale=0.02), wk=normal(hkv * d, hid, scale=0.02),
                 wv=normal(hkv * d, hid, scale=0.02),
                 v_cache=torch.zeros((n + qn, hkv, d), dtype=dt, device=device),
                 k_cache=torch.zeros((n + qn, hkv, d), dtype=dt, device=device))
        L["v_cache"][:n] = normal(n, hkv, d)
        del hidden
        out.append(L)
    return out


# --------------------------------------------------------------------------
# CPU baseline: the oracle as it stands, on a bounded sample
# --------------------------------------------------------------------------

def cpu_baseline(cfg, row_stride=1):
    """Times the CPU oracle on the same seeded workload.  Restore, query
    projection, score and selection run in full; the row-wise steps
    (projection, scatter, attention) run on every `row_stride`-th recomputed
    row and are scaled by the row count."""
    from oracle import pkv_oracle as O          # only this leg touches oracle/
    from threadpoolctl import threadpool_info

    n, qn = cfg.n_ctx, cfg.n_query
    k = synth.select_count(cfg.ratio, n)
    layer = synth.make_layer(cfg, 0)
    geo = dict(n_q_heads=cfg.n_q_heads, n_kv_heads=cfg.n_kv_heads,
               head_dim=cfg.head_dim, theta=cfg.theta)

    def project_q(rows):
        rows = np.asarray(rows)
        return O.project_qkv_rows(layer["hidden"], rows, rows, layer["wq"], layer["wk"],
                                  layer["wv"], dtype=cfg.dtype, **geo)[0]

    synth.plant(cfg, layer, 0, project_q, lambda x, p: O.rope_rotate(x, p, cfg.theta))
    L = {name: v.astype(np.float64) for name, v in layer.items()}
    del layer
    t = {}
    t0 = time.perf_counter()
    k_rope = O.rope_restore(L["k_nope"], np.arange(n), cfg.theta, cfg.dtype)
    t["rope_restore"] = time.perf_counter() - t0
    t0 = time.perf_counter()
    q_rows = np.arange(n, n + qn)
    q_s = O.project_qkv_rows(L["hidden"], q_rows, q_rows, L["wq"], L["wk"], L["wv"],
                             dtype=cfg.dtype, **geo)[0]
    score = O.fuse_score(np.zeros(n), O.query_score(q_s, k_rope))
    t["query_score"] = time.perf_counter() - t0
    t0 = time.perf_counter()
    sel = O.topk_select(score, k)
    t["topk_select"] = time.perf_counter() - t0
    rows = np.concatenate([sel, q_rows])
    sample = rows[::row_stride]
    t0 = time.perf_counter()
    q, k_new, v_new = O.project_qkv_rows(L["hidden"], sample, sample, L["wq"], L["wk"],
                                         L["wv"], dtype=cfg.dtype, **geo)
    t["gather_qkv_proj_sample"] = time.perf_counter() - t0
    t0 = time.perf_counter()
    k_cache = np.zeros((n + qn, cfg.n_kv_heads, cfg.head_dim))
    v_cache = np.zeros_like(k_cache)
    k_cache[:n] = k_rope
    v_cache[:n] = L["v"]
    k_cache, v_cache = O.scatter_kv(k_cache, v_cache, k_new, v_new, sample)
    t["scatter_kv_sample"] = time.perf_counter() - t0
    t0 = time.perf_counter()
    O.sparse_row_attn(q, k_cache, v_cache, sample, dtype=cfg.dtype)
    t["sparse_row_attn_sample"] = time.perf_counter() - t0
    scale = len(rows) / len(sample)
    full = (t["rope_restore"] + t["query_score"] + t["topk_select"] +
            scale * (t["gather_qkv_proj_sample"] + t["sparse_row_attn_sample"]) +
            t["scatter_kv_sample"])
    threads = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    return {
        "value": len(rows) / full, "unit": "tokens/s", "cores": int(threads),
        "kind": "oracle",
        "sample": (f"one layer of {cfg.name}: restore, query projection, score, top-k in full; "
                   f"projection, scatter and attention on " +
                   (f"all {len(rows)} recomputed rows (nothing sampled or scaled); "
                    if row_stride == 1 else
                    f"every {row_stride}th of the {len(rows)} recomputed rows "
                    f"({len(sample)} rows), scaled by {scale:.1f}; ") +
                   f"measured {sum(t.values()):.1f} s of CPU work"),
        "seconds": {name: round(v, 3) for name, v in t.items()},
    }


# --------------------------------------------------------------------------

def attn_flops(rows_pos: np.ndarray, hq: int, d: int) -> float:
    """Causal-masked flops of step 5: QK^T and PV over keys 0..pos inclusive."""
    return 4.0 * hq * d * float((rows_pos.astype(np.int64) + 1).sum())


def time_calls(fn, reps, batch=10):
    """Seconds per call: the median over `reps` batches of `batch` back-to-back calls
    between one pair of events (a single call between events would mostly measure the
    launch gap for the 10-30 us kernels)."""
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    fn()
    torch.cuda.synchronize()
    ts = []
    for _ in range(reps):
        s.record()
        for _ in range(batch):
            fn()
        e.record()
        e.synchronize()
        ts.append(s.elapsed_time(e) * 1e-3 / batch)
    return float(np.median(ts))


def timed_passes(sr, layers, steps):
    """Exactly `steps` passes of the hot path between synchronisations; every
    pkv_sparse_row_attn call inside them is bracketed by events on the launch stream.
    Returns (seconds elapsed, mean seconds per attention call)."""
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(steps * len(layers))]
    orig_attn = api.pkv_sparse_row_attn
    counter = [0]

    def timed_attn(*a, **kw):
        s, e = ev[counter[0]]
        counter[0] += 1
        s.record()
        orig_attn(*a, **kw)
        e.record()
    pipeline.api.pkv_sparse_row_attn = timed_attn
    try:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            sr.run(layers)
        torch.cuda.synchronize()
        elapsed = time.perf_counter() - t0
    finally:
        pipeline.api.pkv_sparse_row_attn = orig_attn
    return elapsed, float(np.mean([s.elapsed_time(e) for s, e in ev])) * 1e-3


def graph_replay_ms(sr, layers, steps):
    """Milliseconds per pass when one pass, captured into a graph, is replayed."""
    cur = torch.cuda.current_stream()
    side = torch.cuda.Stream()          # default priority
    side.wait_stream(cur)
    with torch.cuda.stream(side):
        sr.run(layers)
    cur.wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sr.run(layers)
    graph.replay()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        graph.replay()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) / steps * 1e3
    del graph
    return round(ms, 4)


def extra_workload(name, cfg, device, steps=3, warmup=1, seed=77):
    """One more workload through the same pass, on device-side random draws."""
    layers = random_layers(cfg, device, cfg.n_layers, seed)
    sr = pipeline.SelectiveRecompute(cfg, device)
    for _ in range(warmup):
        sr.run(layers)
    elapsed, t_attn = timed_passes(sr, layers, steps)
    flops = attn_flops(sr.rows.cpu().numpy(), cfg.n_q_heads, cfg.head_dim)
    L = layers[0]
    small = {
        "rope_restore_us": time_calls(lambda: sr.restore(L), 3) * 1e6,
        "query_proj+query_score_us": time_calls(lambda: sr.score_layer(L, False), 3) * 1e6,
        "topk_select_us": time_calls(lambda: sr.select(), 3) * 1e6,
        "gather_qkv_proj_us": time_calls(lambda: api.pkv_gather_qkv_proj(
            sr.lc, L["hidden"], sr.rows, sr.rows, L["wq"], L["wk"], L["wv"], sr.q, sr.k_new,
            sr.v_new, ws=sr.ws), 3, batch=4) * 1e6,
        "scatter_kv_us": time_calls(lambda: api.pkv_scatter_kv(
            sr.lc, sr.k_new, sr.v_new, sr.rows, L["k_cache"], L["v_cache"]), 3) * 1e6,
    }
    per_pass = elapsed / steps
    out = {"workload": name, "n_ctx": cfg.n_ctx, "n_query": cfg.n_query, "ratio": cfg.ratio,
           "rows_recomputed": sr.m, "layers": len(layers),
           "n_score_layers": min(cfg.n_score_layers, len(layers)),
           "ms_per_pass": round(per_pass * 1e3, 4),
           "recomputed_tokens_per_s": round(sr.m * len(layers) / per_pass, 1),
           "sparse_row_attn_us": round(t_attn * 1e6, 1),
           "sparse_row_attn_tflops": round(flops / t_attn / 1e12, 2),
           "sparse_row_attn_frac": round(flops / t_attn / 1e12 / PEAK_BF16_TFLOPS, 4),
           "data": "synthetic (device-side seeded normal draws, nothing planted)"}
    out.update({k: round(v, 1) for k, v in small.items()})
    del layers, sr
    torch.cuda.empty_cache()
    return out


def extras(device):
    """The other workloads of the list: ratios 0.1 / 0.4 at the benchmark shape, the
    8k and the 128k context, and the 32-layer stack with scoring fused over 2 layers at
    three ratios (the hidden states are supplied per layer, as in the timed pass)."""
    c3, c4 = synth.CONFIGS[3], synth.CONFIGS[4]
    todo = [("cfg3-shape r=0.1", c3.with_(ratio=0.1)), ("cfg3-shape r=0.4", c3.with_(ratio=0.4)),
            ("cfg2 8k r=0.2", synth.CONFIGS[2]), ("cfg5 128k r=0.2", synth.CONFIGS[5])]
    todo += [(f"cfg4 32 layers r={r}", c4.with_(ratio=r)) for r in (0.1, 0.2, 0.4)]
    # the first three or four passes after an idle spell run up to 10 % slower than the
    # steady state, so the short single-layer workloads get more warm-up passes
    return [extra_workload(name, cfg, device, steps=2 if cfg.n_layers > 1 else 10,
                           warmup=1 if cfg.n_layers > 1 else 5)
            for name, cfg in todo]


def bandwidth(cfg, device, reps=5):
    """The HBM-bound calls and a plain copy, warm (one buffer set over and over: what fits
    the 256 MB Infinity Cache is served from it) and cold (a rotation over buffer sets whose
    touched bytes add up to more than 512 MB between two visits of the same set)."""
    lc = pipeline.layer_cfg(cfg)
    dt = lc.torch_dtype
    n, qn = cfg.n_ctx, cfg.n_query
    hkv, d, hid = cfg.n_kv_heads, cfg.head_dim, cfg.hidden
    m = synth.select_count(cfg.ratio, n) + qn
    row_b = hkv * d * 2
    rows = torch.sort(torch.randperm(n + qn, device=device)[:m])[0].to(torch.int32)

    def new(*shape):
        return torch.randn(shape, device=device).to(dt)

    w_norm = torch.ones(hid, dtype=dt, device=device)
    calls = {
        "rope_restore": (lambda: (new(n, hkv, d), torch.empty((n, hkv, d), dtype=dt, device=device)),
                         lambda b: api.pkv_rope_restore(lc, b[0], b[1], None, 0),
                         2.0 * n * row_b),
        "scatter_kv": (lambda: (new(m, hkv, d), new(m, hkv, d), new(n + qn, hkv, d),
                                new(n + qn, hkv, d)),
                       lambda b: api.pkv_scatter_kv(lc, b[0], b[1], rows, b[2], b[3]),
                       4.0 * m * row_b),
        "gather_rows": (lambda: (new(n + qn, hid), torch.empty((m, hid), dtype=dt, device=device)),
                        lambda b: api.pkv_gather_rows(b[0], rows, b[1]),
                        2.0 * m * hid * 2),
        "rmsnorm_rows": (lambda: (new(m, hid), torch.empty((m, hid), dtype=dt, device=device)),
                         lambda b: api.pkv_rmsnorm_rows(b[0], None, w_norm, 1e-5, b[1]),
                         2.0 * m * hid * 2),
        "plain_copy_same_bytes_as_rope_restore": (
            lambda: (new(n, hkv, d), torch.empty((n, hkv, d), dtype=dt, device=device)),
            lambda b: b[1].copy_(b[0]), 2.0 * n * row_b),
    }
    out = {}
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for name, (make, call, nbytes) in calls.items():
        n_sets = max(2, int(np.ceil(640e6 / nbytes)) + 1)
        sets = [make() for _ in range(n_sets)]
        for b in sets:
            call(b)
        torch.cuda.synchronize()
        warm = time_calls(lambda: call(sets[0]), reps)
        ts = []
        for _ in range(reps):
            s.record()
            for b in sets:
                call(b)
            e.record()
            e.synchronize()
            ts.append(s.elapsed_time(e) * 1e-3 / n_sets)
        cold = float(np.median(ts))
        out[name] = {"bytes": nbytes, "buffer_sets": n_sets,
                     "warm_us": round(warm * 1e6, 1),
                     "warm_GB/s": round(nbytes / warm / 1e9, 1),
                     "warm_frac": round(nbytes / warm / 1e9 / PEAK_HBM_GBS, 4),
                     "cold_us": round(cold * 1e6, 1),
                     "cold_GB/s": round(nbytes / cold / 1e9, 1),
                     "cold_frac": round(nbytes / cold / 1e9 / PEAK_HBM_GBS, 4)}
        del sets
        torch.cuda.empty_cache()
    big = torch.empty(1 << 30, dtype=torch.uint8, device=device)
    big2 = torch.empty_like(big)
    t = time_calls(lambda: big2.copy_(big), 3, batch=3)
    out["plain_copy_1GiB"] = {"bytes": 2.0 * (1 << 30), "cold_us": round(t * 1e6, 1),
                              "cold_GB/s": round(2.0 * (1 << 30) / t / 1e9, 1),
                              "cold_frac": round(2.0 * (1 << 30) / t / 1e9 / PEAK_HBM_GBS, 4)}
    return out


def diagnostics_report(device, layer, plants, sr):
    """(1) Hit rates of the planted tokens under two criteria at the timed workload: the
    user-query score the pass selected with, and the global column sum of Appendix B,
    Tab. 3 (the attention a token receives from all rows).  (2) Overlap ratios of
    Sec. 3.1 and the chunk-size sweep of Sec. 5.5 on a small random model."""
    from paper_2602_02579_amd import diagnostics
    out = {}
    cfg = sr.cfg
    if plants is not None:
        dg = diagnostics.Diagnostics(cfg, 64, 1e-5, device)
        t0 = time.perf_counter()
        beta = dg.column_sum_from_hidden(layer["hidden"], layer, layer["k_nope"],
                                         layer["v_cache"][:cfg.n_ctx])
        by_colsum = diagnostics.top_indices(beta, sr.k).cpu().numpy()
        torch.cuda.synchronize()
        by_query = sr.rows[:sr.k].cpu().numpy()
        rel, sal = plants["relevant"], plants["salient"]
        out["planted_tokens"] = {
            "workload": cfg.name, "ratio": cfg.ratio,
            "query_relevant_selected": {"query_score": float(np.isin(rel, by_query).mean()),
                                        "global_column_sum": float(np.isin(rel, by_colsum).mean())},
            "globally_salient_selected": {"query_score": float(np.isin(sal, by_query).mean()),
                                          "global_column_sum": float(np.isin(sal, by_colsum).mean())},
            "column_sum_pass_ms": round((time.perf_counter() - t0) * 1e3, 1)}
        del dg, beta
    small = synth.Config("diag-model", "bf16", 8, 256, 32, 8, 2, 128, 1024, 500000.0, seed=31,
                         n_layers=4, n_score_layers=4)
    inter = 2048
    dt = torch.bfloat16
    embed = torch.from_numpy(synth.make_embed(small)).to(dt).to(device)
    blocks = [{k: torch.from_numpy(v).to(dt).to(device)
               for k, v in synth.make_block_weights(small, li, inter).items()}
              for li in range(small.n_layers)]
    dg = diagnostics.Diagnostics(small, inter, 1e-5, device)
    ratios = [0.1, 0.2, 0.4]
    sweep = {}
    for chunk_len in (64, 128, 256, 512, 2048):
        res = dg.selection_diagnostics(embed, blocks, chunk_len, ratios)
        sweep[str(chunk_len)] = {name: [round(x, 4) for x in res[name]]
                                 for name in ("fused", "first_layer", "column_sum")}
    out["overlap_with_full_prefill_query_attention"] = {
        "model": "4 random layers, 2048 context tokens, 32 query tokens, 8/2 heads, hidden 1024",
        "ratios": ratios, "by_chunk_len": sweep}
    return out


def carried_model(cfg, device, n_layers, inter=14336, eps=1e-5, steps=3):
    """One pass = Stage I (query rows, 2 scoring layers) + Stage II (selected + query
    rows, every layer) with attention and MLP in every layer.  Weights and caches are
    seeded device-side normal draws (unit-scale outputs); nothing is planted, the
    selection is whatever the random scores give."""
    cfg = cfg.with_(n_layers=n_layers, n_score_layers=min(2, n_layers))
    lc = pipeline.layer_cfg(cfg)
    dt = lc.torch_dtype
    gen = torch.Generator(device=device)
    gen.manual_seed(1234 + cfg.seed)
    hq, hkv, d, hid = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.hidden
    n, qn = cfg.n_ctx, cfg.n_query

    def normal(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=device) * scale).to(dt)

    layers = []
    for _ in range(n_layers):
        L = dict(k_nope=normal(n, hkv, d), k_cache=torch.zeros((n + qn, hkv, d), dtype=dt,
                                                               device=device),
                 v_cache=torch.zeros((n + qn, hkv, d), dtype=dt, device=device),
                 w_in=torch.ones(hid, dtype=dt, device=device),
                 w_post=torch.ones(hid, dtype=dt, device=device),
                 wq=normal(hq * d, hid, scale=1.5 * hid ** -0.5),
                 wk=normal(hkv * d, hid, scale=1.5 * hid ** -0.5),
                 wv=normal(hkv * d, hid, scale=hid ** -0.5),
                 wo=normal(hid, hq * d, scale=(hq * d) ** -0.5),
                 w_gate=normal(inter, hid, scale=1.5 * hid ** -0.5),
                 w_up=normal(inter, hid, scale=hid ** -0.5),
                 w_down=normal(hid, inter, scale=inter ** -0.5))
        L["v_cache"][:n] = normal(n, hkv, d)
        layers.append(L)
    embed = normal(n + qn, hid)
    cr = model.CarriedRows(cfg, inter, eps, device)
    # Stage II writes the recomputed values into v_cache: every timed pass starts from the
    # assembled chunk values again (copied back outside the timed interval), so each one is
    # the first-pass problem; the keys are restored from k_nope by the pass itself
    pristine = [L["v_cache"].clone() for L in layers]
    per_pass = []
    sel = []
    for it in range(steps + 1):                 # the first pass warms up
        for L, v0 in zip(layers, pristine):
            L["v_cache"].copy_(v0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        h = cr.run(embed, layers)
        torch.cuda.synchronize()
        if it:
            per_pass.append(time.perf_counter() - t0)
        sel.append(cr.rows.clone())
    per_pass = float(np.median(per_pass))
    same_selection = all(torch.equal(sel[0], x) for x in sel[1:])
    del pristine
    finite = bool(torch.isfinite(h.float()).all())
    # the glue calls of one Stage II layer, one by one
    m = cr.m
    L = layers[0]
    x, hbuf, g, attn = cr.x[:m], cr.h[:m], cr.g[:m], cr.attn[:m].view(m, -1)
    calls = {
        "rmsnorm_rows": (lambda: api.pkv_rmsnorm_rows(hbuf, None, L["w_in"], eps, x),
                         2.0 * m * hid * 2, "hbm"),
        "o_proj+residual": (lambda: api.pkv_linear_rows(attn, L["wo"], hbuf, hbuf, ws=cr.ws),
                            2.0 * m * hid * hq * d, "mfma"),
        "swiglu_rows": (lambda: api.pkv_swiglu_rows(x, L["w_gate"], L["w_up"], g, ws=cr.ws),
                        4.0 * m * hid * inter, "mfma"),
        "down_proj+residual": (lambda: api.pkv_linear_rows(g, L["w_down"], hbuf, hbuf,
                                                           ws=cr.ws),
                               2.0 * m * hid * inter, "mfma"),
    }
    glue = {}
    for name, (fn, work, bound) in calls.items():
        t = time_calls(fn, 5, batch=4)
        glue[name] = {"us": round(t * 1e6, 1), "bound": bound}
        if bound == "hbm":
            glue[name]["GB/s"] = round(work / t / 1e9, 1)
            glue[name]["frac"] = round(work / t / 1e9 / PEAK_HBM_GBS, 4)
        else:
            glue[name]["TFLOP/s"] = round(work / t / 1e12, 2)
            glue[name]["frac"] = round(work / t / 1e12 / PEAK_BF16_TFLOPS, 4)
    # the scoring work of one Stage I layer on the query rows, both ways: attention that
    # also emits the context-only normaliser + one column-sum pass, against the two-pass
    # score + plain attention
    stage1 = None
    if cr.fuse_stage1:
        q1, a1 = cr.q[:qn], cr.attn[:qn]
        kc, vc = L["k_cache"], L["v_cache"]

        def fused():
            api.pkv_sparse_row_attn_ctx_lse(lc, q1, kc, vc, cr.q_rows, a1, None, cr.lse_ctx, n,
                                            ws=cr.ws)
            api.pkv_query_score_lse(lc, q1, kc[:n], cr.lse_ctx, None, cr.score,
                                    accumulate=False, ws=cr.ws)

        def two_calls():
            api.pkv_query_score(lc, q1, kc[:n], cr.score, accumulate=False, ws=cr.ws)
            api.pkv_sparse_row_attn(lc, q1, kc, vc, cr.q_rows, a1, None, ws=cr.ws)
        stage1 = {"fused_us": round(time_calls(fused, 5) * 1e6, 1),
                  "score_then_attention_us": round(time_calls(two_calls, 5) * 1e6, 1),
                  "what": "query-row attention + score of one scoring layer (128 rows, 32k keys)"}
    return {"layers": n_layers, "n_score_layers": cfg.n_score_layers, "mlp_width": inter,
            "stage1_scoring_layer": stage1,
            "rows_stage2": m, "rows_stage1": qn, "ms_per_pass": round(per_pass * 1e3, 3),
            "ms_per_layer_stage2_est": round(sum(v["us"] for v in glue.values()) * 1e-3, 3),
            "recomputed_tokens_per_s": round(m * n_layers / per_pass, 1),
            "output_finite": finite, "same_selection_every_pass": same_selection,
            "fused_stage1": cr.fuse_stage1,
            # a whole run scores its last scoring layer without the attention
            "fused_scoring_layers": cfg.n_score_layers - 1 if cr.fuse_stage1 else 0,
            "data": "synthetic (device-side seeded normal draws)",
            "glue": glue}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--profile-call", default=None,
                    help="run the whole path once, then only this call --reps times and "
                         "exit (for rocprofv3 counter runs): rope_restore, query_score, "
                         "topk_select, gather_qkv_proj, scatter_kv, sparse_row_attn; or "
                         "copy = a plain 1 GiB device copy that calibrates the HBM counters")
    ap.add_argument("--reps", type=int, default=3)
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the other workloads, the cold/warm bandwidth table and the "
                         "diagnostics")
    ap.add_argument("--model-layers", type=int, default=4,
                    help="layers of the carried-hidden-state model timed after the steps "
                         "(0 = skip); bf16 configurations with head_dim 128 only")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        sys.exit("bench.py: this build runs on ONE GPU only (no collectives, no sharding); "
                 "run with --gpus 1")
    if not torch.cuda.is_available():
        sys.exit("bench.py needs a GPU")
    api.load_library()           # fails loudly if libpkv.so is missing
    device = torch.device("cuda:0")
    torch.cuda.set_device(device)
    cfg = synth.CONFIGS[args.config]
    layers, plants = build_gpu_workload(cfg, device)
    sr = pipeline.SelectiveRecompute(cfg, device)

    for _ in range(args.warmup):
        sr.run(layers)
    torch.cuda.synchronize()

    if args.profile_call:
        L0 = layers[0]
        cal_src = torch.empty(1 << 30, dtype=torch.uint8, device=device)
        cal_dst = torch.empty_like(cal_src)
        one = {
            "copy": lambda: cal_dst.copy_(cal_src),
            "rope_restore": lambda: sr.restore(L0),
            "query_score": lambda: sr.score_layer(L0, False),
            "topk_select": lambda: sr.select(),
            "gather_qkv_proj": lambda: api.pkv_gather_qkv_proj(
                sr.lc, L0["hidden"], sr.rows, sr.rows, L0["wq"], L0["wk"], L0["wv"], sr.q,
                sr.k_new, sr.v_new, ws=sr.ws),
            "scatter_kv": lambda: api.pkv_scatter_kv(sr.lc, sr.k_new, sr.v_new, sr.rows,
                                                     L0["k_cache"], L0["v_cache"]),
            "sparse_row_attn": lambda: api.pkv_sparse_row_attn(
                sr.lc, sr.q, L0["k_cache"], L0["v_cache"], sr.rows, sr.out, sr.lse, ws=sr.ws),
        }[args.profile_call]
        one()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(args.reps):
            one()
        e1.record()
        torch.cuda.synchronize()
        print(json.dumps({"profiled_call": args.profile_call, "reps": args.reps,
                          "workload": cfg.name,
                          "us_per_call": round(e0.elapsed_time(e1) * 1e3 / args.reps, 1)}))
        return

    # ---- timed region: exactly K steps; the dominant kernel (step 5) is
    # bracketed by events on the launch stream inside it ---------------------
    elapsed, t_attn = timed_passes(sr, layers, args.steps)

    ms_per_step = elapsed / args.steps * 1e3
    m_rows = sr.m * len(layers)
    value = m_rows / (elapsed / args.steps)
    rows_pos = sr.rows.cpu().numpy()
    flops = attn_flops(rows_pos, cfg.n_q_heads, cfg.head_dim)
    peak = PEAK_BF16_TFLOPS if cfg.dtype == "bf16" else PEAK_F32_TFLOPS
    achieved = flops / t_attn / 1e12

    # ---- per-call breakdown (outside the timed region) ---------------------
    L = layers[0]
    elt = 2 if cfg.dtype == "bf16" else 4
    row_b = cfg.n_kv_heads * cfg.head_dim * elt
    calls = {
        "rope_restore": (lambda: sr.restore(L), 2.0 * cfg.n_ctx * row_b, "hbm"),
        "query_proj+query_score": (lambda: sr.score_layer(L, False),
                                   2.0 * cfg.n_q_heads * cfg.n_query * cfg.n_ctx * cfg.head_dim,
                                   "mfma"),
        "topk_select": (lambda: sr.select(), 4.0 * cfg.n_ctx + 4.0 * sr.k, "hbm"),
        "gather_qkv_proj": (lambda: api.pkv_gather_qkv_proj(
            sr.lc, L["hidden"], sr.rows, sr.rows, L["wq"], L["wk"], L["wv"], sr.q,
            sr.k_new, sr.v_new, ws=sr.ws),
            2.0 * sr.m * cfg.hidden * (cfg.n_q_heads + 2 * cfg.n_kv_heads) * cfg.head_dim,
            "mfma"),
        "scatter_kv": (lambda: api.pkv_scatter_kv(sr.lc, sr.k_new, sr.v_new, sr.rows,
                                                  L["k_cache"], L["v_cache"]),
                       4.0 * sr.m * row_b, "hbm"),
        "sparse_row_attn": (lambda: api.pkv_sparse_row_attn(
            sr.lc, sr.q, L["k_cache"], L["v_cache"], sr.rows, sr.out, sr.lse, ws=sr.ws),
            flops, "mfma"),
    }
    breakdown = {}
    for name, (fn, work, bound) in calls.items():
        t = time_calls(fn, 10)
        entry = {"us": round(t * 1e6, 1), "bound": bound}
        if bound == "hbm":
            entry["GB/s"] = round(work / t / 1e9, 1)
            entry["frac"] = round(work / t / 1e9 / PEAK_HBM_GBS, 4)
        else:
            entry["TFLOP/s"] = round(work / t / 1e12, 2)
            entry["frac"] = round(work / t / 1e12 / peak, 4)
        breakdown[name] = entry

    result = {
        "metric": (f"recomputed tokens/s (selective-recompute hot path, "
                   f"{cfg.n_ctx // 1024}k ctx, r={cfg.ratio})"),
        "value": round(value, 1), "unit": "tokens/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None,
        "dtype": cfg.dtype, "data": "synthetic",
        "config": {"workload": cfg.name, "n_ctx": cfg.n_ctx, "n_query": cfg.n_query,
                   "chunks": f"{cfg.n_chunks}x{cfg.chunk_len}", "ratio": cfg.ratio,
                   "k": sr.k, "rows_recomputed": sr.m, "layers": len(layers),
                   "n_score_layers": min(cfg.n_score_layers, len(layers)),
                   "heads": f"{cfg.n_q_heads}/{cfg.n_kv_heads}", "head_dim": cfg.head_dim,
                   "hidden": cfg.hidden},
        "context_tokens_per_s": round(cfg.n_ctx * len(layers) / (elapsed / args.steps), 1),
        "sparse_row_attn_tflops": round(achieved, 2),
        "roofline": {"kernel": "pkv_sparse_row_attn", "bound": "mfma",
                     "achieved": round(achieved, 3), "peak": peak, "unit": "TFLOP/s",
                     "frac": round(achieved / peak, 4),
                     "traffic": MEASURED_ATTN_TRAFFIC_BYTES.get(cfg.name),
                     "traffic_source": TRAFFIC_SOURCE,
                     "flops_per_launch": flops, "avg_launch_s": t_attn,
                     "launch": "pkv_sparse_row_attn = a first kernel (a V^T copy that also clears the "
                               "work counters; with fewer rows the clear alone) + "
                               "attn_w8n_kernel, timed with events on the launch stream"},
        "breakdown": breakdown,
    }
    # the same pass with steps 4a + 4b fused into one call (outside `value`)
    sr_f = pipeline.SelectiveRecompute(cfg, device, fused_scatter=True)
    sr_f.run(layers)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        sr_f.run(layers)
    torch.cuda.synchronize()
    result["ms_per_step_fused_cache_update"] = round(
        (time.perf_counter() - t0) / args.steps * 1e3, 4)
    def section(key, fn):
        """The sections below are outside `value`: one that fails (memory, an unsupported
        shape) says so in its place and the line is still printed."""
        try:
            result[key] = fn()
        except Exception as exc:   # noqa: BLE001
            result[key] = {"error": f"{type(exc).__name__}: {exc}"}
            torch.cuda.synchronize()
            torch.cuda.empty_cache()

    if not args.no_extras:
        # the same two passes replayed from a captured graph: what is left of the launch
        # gaps between the small kernels at the head of a pass (outside `value`, whose timed
        # region carries the events of the roofline and is launched call by call)
        section("ms_per_step_graph_replay", lambda: graph_replay_ms(sr, layers, args.steps))
        section("ms_per_step_fused_cache_update_graph_replay",
                lambda: graph_replay_ms(sr_f, layers, args.steps))
    del sr_f
    if not args.no_extras and cfg.dtype == "bf16":
        section("diagnostics", lambda: diagnostics_report(device, layers[0], plants, sr))
    del layers, sr
    torch.cuda.empty_cache()
    if not args.no_extras and cfg.dtype == "bf16":
        section("bandwidth", lambda: bandwidth(cfg, device))
        section("extras", lambda: extras(device))
    if args.model_layers > 0 and cfg.dtype == "bf16":
        section("carried_model",
                lambda: carried_model(cfg.with_(n_layers=1), device, args.model_layers))
    if not args.no_cpu_baseline:
        section("cpu_baseline",
                lambda: cpu_baseline(cfg.with_(n_layers=1, n_score_layers=1)))
    print(json.dumps(result))


if __name__ == "__main__":
    main()
