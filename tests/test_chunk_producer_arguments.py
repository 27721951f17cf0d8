"""The host side of the chunk producer: what it refuses before any library call, the rows, positions
and scratch that it hands to the calls, and the buffers that it keeps."""

import os

import pytest
import torch

from paper_2602_02579_amd import api, diagnostics
from tests.test_gpu_model import CASES, EPS


def producer():
    cfg, inter = CASES[sorted(CASES)[0]]
    device = torch.device("cpu")
    dg = diagnostics.Diagnostics(cfg, inter, EPS, device)
    return dg, torch.zeros((cfg.n_ctx, cfg.hidden), dtype=dg.dt)


@pytest.mark.parametrize("chunk_len", [0, -1, -512])
def test_chunk_lengths_that_give_no_chunk_are_refused(chunk_len):
    dg, embed = producer()
    with pytest.raises(ValueError):
        dg.chunk_isolated_cache(embed, [{}], chunk_len)


def test_chunks_of_one_token_are_refused():
    dg, embed = producer()
    with pytest.raises(ValueError, match="at least two tokens"):
        dg.chunk_isolated_cache(embed, [{}], 1)


def kept_bytes(dg):
    held, seen = {}, [dg.__dict__]
    while seen:
        x = seen.pop()
        if isinstance(x, torch.Tensor):
            held[x.untyped_storage().data_ptr()] = x.untyped_storage().nbytes()
        elif isinstance(x, dict):
            seen += x.values()
        elif isinstance(x, (list, tuple)):
            seen += x
        elif type(x).__module__.startswith("paper_") and hasattr(x, "__dict__"):
            seen.append(x.__dict__)
    return sum(held.values())


def without_kernels(monkeypatch, calls):
    """The library's calls of the producer, noted instead of made."""
    for name in ("pkv_gather_rows", "pkv_layer_rows", "pkv_rope_restore_layers"):
        monkeypatch.setattr(diagnostics.api, name,
                            lambda *a, _name=name, **kw: calls.append((_name, a, kw)))


@pytest.mark.parametrize("name", ["f32-small", "bf16-tiles"])
def test_what_is_kept_does_not_grow_with_the_lengths_seen(monkeypatch, name):
    """Rows for the longest group of chunks, and no more than as many again for shorter ones, however
    many document and chunk lengths one object prefills."""
    if not os.path.exists(api.library_path()):
        pytest.skip("libpkv.so not built")
    cfg, inter = CASES[name]
    cfg = cfg.with_(n_chunks=1, chunk_len=4000)
    without_kernels(monkeypatch, [])
    cpu = torch.device("cpu")
    longest = diagnostics.Diagnostics(cfg, inter, EPS, cpu)
    embed = torch.zeros((cfg.n_ctx, cfg.hidden), dtype=longest.dt)
    longest.chunk_isolated_cache(embed, [{}], 4000)
    dg = diagnostics.Diagnostics(cfg, inter, EPS, cpu)
    for n in range(4000, 20, -199):
        dg.prefill_cache(embed[:n], [{}])
    lengths = (4000, 17, 100, 334, 512, 1999)
    for chunk_len in lengths:
        dg.chunk_isolated_cache(embed, [{}], chunk_len)
    # shorter sets have fewer rows, but up to as much room for partial sums; and the positions
    # inside chunks of a length are two int32 a row
    scratch = api.pkv_glue_workspace_bytes(dg.dt, 1024, cfg.hidden, cfg.hidden)
    assert kept_bytes(dg) <= 2 * kept_bytes(longest) + 2 * scratch + 8 * 4096 * len(lengths)


@pytest.mark.parametrize("n,chunk_len", [(900, 1000), (1000, 1000), (1000, 300), (700, 64),
                                         (258, 256), (512, 256)])
def test_rows_know_their_cache_row_and_their_place_in_the_chunk(monkeypatch, n, chunk_len):
    if not os.path.exists(api.library_path()):
        pytest.skip("libpkv.so not built")
    cfg, inter = CASES[sorted(CASES)[0]]
    calls = []
    without_kernels(monkeypatch, calls)
    monkeypatch.setattr(diagnostics, "GROUP_ROWS", 512)
    dg = diagnostics.Diagnostics(cfg.with_(n_chunks=1, chunk_len=n), inter, EPS,
                                 torch.device("cpu"))
    embed = torch.zeros((n, cfg.hidden), dtype=dg.dt)
    done = 0
    dg.chunk_isolated_cache(embed, [{}, {}], chunk_len)
    for name, a, kw in calls:
        if name == "pkv_layer_rows":
            m, pos, dst = a[6], a[11], a[12]
            assert torch.equal(dst, torch.arange(m, dtype=torch.int32))
            assert torch.equal(pos, dst % chunk_len)
            assert min(kw["chunk_len"], m) == min(chunk_len, m)
            assert a[9].shape[0] == m and all(t.shape[0] >= m for t in a[1:6])
            need = [api.pkv_chunk_attn_workspace_bytes(dg.lc, m, chunk_len),
                    api.pkv_workspace_bytes(api.CALL_GATHER_QKV_PROJ, dg.lc, 0, m)] + [
                api.pkv_glue_workspace_bytes(dg.dt, m, *s) for s in (
                    (cfg.n_q_heads * cfg.head_dim, cfg.hidden), (cfg.hidden, inter),
                    (inter, cfg.hidden))]
            assert a[14].numel() >= max(need)
        elif name == "pkv_rope_restore_layers":
            assert torch.equal(a[3], -(torch.arange(a[1][0].shape[0], dtype=torch.int32)
                                       % chunk_len))
            done += a[1][0].shape[0]
    assert done == n
