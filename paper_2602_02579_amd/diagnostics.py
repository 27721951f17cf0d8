"""Selection diagnostics of the paper on synthetic models, through the C ABI.

Orchestration only, like ``pipeline`` and ``model``: torch buffers and sequences of
library calls; the set arithmetic of the overlap ratio is host bookkeeping on the
downloaded index lists.

* ``chunk_isolated_cache`` / ``full_prefill_cache``: the producer of the method's input
  (Sec. 2: every chunk is prefilled by itself and its keys are stored without
  positions) and the ordinary prefill it stands in for.  A prefill of T tokens is Stage II
  of the carried-rows model with every row selected; the chunks of a document pass through
  the layers together, each attending within itself.
* ``query_attention_score``: the fused user-query attention to the context (Algorithm 1,
  first stage) over given caches - ProphetKV's criterion on the chunk caches, the ground
  truth G of Sec. 3.1 (Fig. 2) on the full-prefill ones.
* ``column_sum_score``: the attention every context token receives from ALL rows of the
  prompt at one layer (Appendix B, Tab. 3, first factor of the KVShare row), the
  criterion whose budget the globally salient tokens crowd (Sec. 3.1).
* ``overlap_ratio``: |S n G| / |G|.
"""

from __future__ import annotations

from typing import Dict, List, Optional, Sequence, Tuple

import numpy as np
import torch

from . import api
from .model import BLOCK_WEIGHTS, VARIANT_WEIGHTS, CarriedRows
from .pipeline import layer_cfg
from .synth import Config, select_count

Block = Dict[str, torch.Tensor]


def overlap_ratio(selected: torch.Tensor, ground_truth: torch.Tensor) -> float:
    """|S n G| / |G| of two index tensors (Sec. 3.1)."""
    s = np.unique(selected.detach().cpu().numpy())
    g = np.unique(ground_truth.detach().cpu().numpy())
    if g.size == 0:
        raise ValueError("empty ground-truth set")
    return float(np.intersect1d(s, g).size) / float(g.size)


def top_indices(score: torch.Tensor, k: int) -> torch.Tensor:
    idx = torch.empty(k, dtype=torch.int32, device=score.device)
    api.pkv_topk_select(score, k, idx)
    return idx


# Chunks that pass through the layers together hold at most this many rows (one chunk may hold
# more): the linear layers of 8192 rows fill the chip many times over and read the weights once
# where 16 chunks of 512 read them 16 times; further rows only grow the buffers (0.6 GB at 4096 /
# 14336 bf16).  16k tokens in chunks of 512 through two layers of 4096 / 14336, chunk by chunk ->
# 2048 / 8192 / 16384 rows at once: 10.0 -> 6.8 / 5.8 / 5.8 ms; in chunks of 256 through four of
# 1024 / 2048, where 64 chunks made 2000 small launches: 18.1 -> 2.5 / 1.5 / 1.3 ms.
GROUP_ROWS = 8192


class Diagnostics:
    """Work buffers for one model geometry (``cfg``: context, query and head sizes; the
    block weights are passed to the methods as lists of device tensors)."""

    def __init__(self, cfg: Config, inter: int, eps: float, device: torch.device):
        self.cfg, self.inter, self.eps, self.device = cfg, int(inter), float(eps), device
        self.lc = layer_cfg(cfg)
        self.dt = self.lc.torch_dtype
        self._prefill: Dict[int, CarriedRows] = {}   # by rows, rounded up: _prefill_rows
        self._stage1: Optional[CarriedRows] = None

    def _cache_pair(self, rows: int) -> Tuple[torch.Tensor, torch.Tensor]:
        shape = (rows, self.cfg.n_kv_heads, self.cfg.head_dim)
        return (torch.zeros(shape, dtype=self.dt, device=self.device),
                torch.zeros(shape, dtype=self.dt, device=self.device))

    # ---- producers -------------------------------------------------------------------
    def prefill_cache(self, embed_rows: torch.Tensor,
                      blocks: Sequence[Block]) -> Tuple[List[torch.Tensor], List[torch.Tensor]]:
        """Ordinary causal prefill of ``embed_rows [T, hid]`` at positions 0..T-1; returns
        per layer the keys in their stored, position-free form and the values."""
        shape = (embed_rows.shape[0], self.cfg.n_kv_heads, self.cfg.head_dim)
        k, v = ([torch.empty(shape, dtype=self.dt, device=self.device) for _ in blocks]
                for _ in range(2))
        self._check_chunk(shape[0])
        self._prefill_into(embed_rows, blocks, k, v, shape[0])
        return k, v

    @staticmethod
    def _check_chunk(tokens: int) -> None:
        if tokens < 2:
            raise ValueError("a chunk needs at least two tokens")

    # Buffers for t rows: kept by a power of two of rows, from 1024 on, so that whatever lengths an
    # object is given it keeps less than twice the rows of the largest set (a set for each length
    # would grow without end, and one set that grows would give memory back that work on another
    # stream or a captured graph still uses).  A set is its rows of h, x, q, attn and g, and up to
    # 67 MB of scratch for partial sums.  Row i is cache row i; -positions turn keys back.
    def _prefill_rows(self, t: int) -> CarriedRows:
        rows = max(1024, 1 << (t - 1).bit_length())
        cr = self._prefill.get(rows)
        if cr is None:   # every row recomputed: all but one "selected" and one closing row
            sub = self.cfg.with_(n_chunks=1, chunk_len=rows - 1, n_query=1)
            cr = CarriedRows(sub, self.inter, self.eps, self.device, k=rows - 1)
            cr.rows[:rows - 1] = torch.arange(rows - 1, dtype=torch.int32, device=self.device)
            cr.in_chunks = {}   # chunk length (0: one chunk) -> positions in it, and their negatives
            cr.views = {}       # (t, chunk length) -> what a call takes of the buffers
            self._prefill[rows] = cr
        return cr

    # the same for chunks of chunk_len tokens, the last one with what is left, into given tensors:
    # every one of their T rows is written before anything reads it, and the inverse rotation runs
    # in place
    def _prefill_into(self, embed_rows: torch.Tensor, blocks: Sequence[Block],
                      k: List[torch.Tensor], v: List[torch.Tensor], chunk_len: int) -> None:
        t = embed_rows.shape[0]
        cr = self._prefill_rows(t)
        if (t, chunk_len) not in cr.views:
            if len(cr.views) == 64:   # views are cheap to make again
                cr.views.clear()
            length = chunk_len if t > chunk_len else 0
            if length not in cr.in_chunks:
                inside = cr.rows % length if length else cr.rows
                cr.in_chunks[length] = inside, -inside
            pos, neg_pos = cr.in_chunks[length]
            cr.views[t, chunk_len] = (
                cr.h[:t], cr.rows[:t], pos[:t], neg_pos[:t],
                api.pkv_chunk_attn_workspace_bytes(self.lc, t, chunk_len))
        h, rows, pos, neg_pos, need = cr.views[t, chunk_len]
        # the layers' scratch is largest with all rows of the set; the attention's depends on the
        # chunks and may be more
        ws = cr.ws if need <= cr.ws.numel() else torch.empty(need, dtype=torch.uint8,
                                                             device=self.device)
        api.pkv_gather_rows(embed_rows.contiguous(), rows, h)
        for li, b in enumerate(blocks):   # the last one stops at its cache rows
            L = {name: b[name] for name in BLOCK_WEIGHTS + VARIANT_WEIGHTS if name in b}
            L["k_cache"], L["v_cache"] = k[li], v[li]
            cr._layer(L, pos, t, score=None, caches_only=li == len(blocks) - 1,
                      chunks=(rows, chunk_len), ws=ws)
        api.pkv_rope_restore_layers(self.lc, k, k, neg_pos)   # inverse rotation

    def chunk_isolated_cache(self, embed: torch.Tensor, blocks: Sequence[Block],
                             chunk_len: int):
        """Per-layer ``(k_nope, v) [n_ctx, Hkv, D]`` with every chunk prefilled alone."""
        n = self.cfg.n_ctx
        starts = range(0, n, chunk_len)
        if blocks and not starts:
            raise ValueError(f"no chunks of {chunk_len} tokens in {n}")
        shape = (n, self.cfg.n_kv_heads, self.cfg.head_dim)
        ks, vs = ([torch.empty(shape, dtype=self.dt, device=self.device) for _ in blocks]
                  for _ in range(2))
        end = 0
        for a in starts:
            end = a + embed[a:min(a + chunk_len, n)].shape[0]
            self._check_chunk(end - a)
        group = max(1, GROUP_ROWS // chunk_len) * chunk_len
        for a in range(0, end, group):   # straight into the group's rows of the whole
            b = min(a + group, end)
            self._prefill_into(embed[a:b], blocks, [x[a:b] for x in ks], [x[a:b] for x in vs],
                               chunk_len)
        return [x[:end] for x in ks], [x[:end] for x in vs]

    def full_prefill_cache(self, embed: torch.Tensor, blocks: Sequence[Block]):
        return self.chunk_isolated_cache(embed, blocks, self.cfg.n_ctx)

    # ---- criteria --------------------------------------------------------------------
    def _layers_with_cache(self, blocks, k_nope, v):
        n, qn = self.cfg.n_ctx, self.cfg.n_query
        layers = []
        for li, b in enumerate(blocks):
            L = {name: b[name] for name in BLOCK_WEIGHTS + VARIANT_WEIGHTS if name in b}
            L["k_nope"] = k_nope[li]
            L["k_cache"], L["v_cache"] = self._cache_pair(n + qn)
            L["v_cache"][:n] = v[li]
            layers.append(L)
        return layers

    def query_attention_score(self, embed: torch.Tensor, blocks: Sequence[Block],
                              k_nope, v, n_score_layers: int) -> torch.Tensor:
        """Fused Stage I score of the user-query rows over the given per-layer caches."""
        if self._stage1 is None:
            self._stage1 = CarriedRows(self.cfg, self.inter, self.eps, self.device, k=0)
        cr = self._stage1
        layers = self._layers_with_cache(blocks[:n_score_layers], k_nope, v)
        cr.stage1(embed, layers, n_score_layers)
        return cr.score.clone()

    def column_sum_score(self, embed: torch.Tensor, block: Block, k_nope: torch.Tensor,
                         v: torch.Tensor) -> torch.Tensor:
        """Attention received by every context token from all prompt rows at the layer
        ``block`` whose (normalised) input rows are RMSNorm(embed) - the first layer."""
        n, qn = self.cfg.n_ctx, self.cfg.n_query
        x = torch.empty_like(embed)
        api.pkv_rmsnorm_rows(embed, None, block["w_in"], self.eps, x)
        return self.column_sum_from_hidden(x, block, k_nope, v)

    def column_sum_from_hidden(self, hidden: torch.Tensor, w: Block, k_nope: torch.Tensor,
                               v: torch.Tensor) -> torch.Tensor:
        """The same with the layer's input rows ``hidden [n_ctx + n_query, hid]`` supplied
        (``w`` holds ``wq, wk, wv``): context keys are the restored chunk keys, the query
        rows' keys are projected; every row attends causally over that cache."""
        cfg, lc = self.cfg, self.lc
        n, qn = cfg.n_ctx, cfg.n_query
        t = n + qn
        dev = self.device
        pos = torch.arange(t, dtype=torch.int32, device=dev)
        k_cache, v_cache = self._cache_pair(t)
        v_cache[:n] = v
        api.pkv_rope_restore(lc, k_nope, k_cache[:n], None, 0)
        q = torch.empty((t, cfg.n_q_heads, cfg.head_dim), dtype=self.dt, device=dev)
        ws = torch.empty(max(api.pkv_workspace_bytes(api.CALL_GATHER_QKV_PROJ, lc, 0, t),
                             api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, lc, t, t),
                             api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, lc, t, t), 256),
                         dtype=torch.uint8, device=dev)
        variant = {name: w[name] for name in VARIANT_WEIGHTS if name in w}
        api.pkv_gather_qkv_proj_ex(lc, hidden, None, pos, w["wq"], None, None, q, None, None,
                                   ws=ws, norm_eps=self.eps, **variant)
        q_tail = torch.empty((qn, cfg.n_q_heads, cfg.head_dim), dtype=self.dt, device=dev)
        api.pkv_gather_qkv_proj_scatter(lc, hidden, pos[n:], pos[n:], w["wq"], w["wk"], w["wv"],
                                        q_tail, k_cache, v_cache, pos[n:], ws=ws,
                                        norm_eps=self.eps, **variant)
        out = torch.empty_like(q)
        lse = torch.empty((t, cfg.n_q_heads), dtype=torch.float32, device=dev)
        api.pkv_sparse_row_attn(lc, q, k_cache, v_cache, pos, out, lse, ws=ws)
        beta = torch.empty(t, dtype=torch.float32, device=dev)
        api.pkv_query_score_lse(lc, q, k_cache, lse, pos, beta, accumulate=False, ws=ws)
        return beta[:n].clone()

    # ---- the tables ------------------------------------------------------------------
    def selection_diagnostics(self, embed: torch.Tensor, blocks: Sequence[Block],
                              chunk_len: int, ratios: Sequence[float]):
        """Overlap with the full-prefill ground truth (Sec. 3.1) of the fused
        query-attention criterion, its first-layer-only form (Sec. 4.3) and the global
        column sum of the first layer (Appendix B), at each selection ratio."""
        n = self.cfg.n_ctx
        n_layers = len(blocks)
        kc, vc = self.chunk_isolated_cache(embed, blocks, chunk_len)
        kf, vf = self.full_prefill_cache(embed, blocks)
        scores = dict(
            truth=self.query_attention_score(embed, blocks, kf, vf, n_layers),
            fused=self.query_attention_score(embed, blocks, kc, vc, n_layers),
            first_layer=self.query_attention_score(embed, blocks, kc, vc, 1),
            column_sum=self.column_sum_score(embed, blocks[0], kc[0], vc[0]))
        out = dict(fused=[], first_layer=[], column_sum=[], scores=scores)
        for r in ratios:
            k = select_count(r, n)
            g = top_indices(scores["truth"], k)
            for name in ("fused", "first_layer", "column_sum"):
                out[name].append(overlap_ratio(top_indices(scores[name], k), g))
        return out
