"""Both stages of ProphetKV with the hidden states carried through the layers.

Orchestration only, like ``pipeline``: preallocated torch buffers and the sequence
of C-ABI calls.  Stage I (Sec. 4.2) runs the user-query rows alone through the
first ``n_score_layers`` layers against the imprecise cache and accumulates their
attention to the context; Stage II (Sec. 4.3, Appendix E) runs the selected and the
query rows through every layer, replacing their cache rows before they attend.
Between the hot-path calls the rows pass through the rest of a pre-norm decoder
block (RMSNorm, output projection + residual, gated MLP + residual) - the public
Llama block of the models the paper evaluates (Sec. 5.1).
"""

from __future__ import annotations

from typing import Dict, List, Optional

import numpy as np
import torch

from . import api
from .pipeline import layer_cfg, restore_together
from .synth import Config, select_count

BLOCK_WEIGHTS = ("w_in", "wq", "wk", "wv", "wo", "w_post", "w_gate", "w_up", "w_down")
# block variants of the other public model families the paper evaluates (Sec. 5.1):
# projection biases (Qwen2.5) and per-head RMS-norm gains of Q and K (Qwen3)
VARIANT_WEIGHTS = ("bq", "bk", "bv", "q_norm", "k_norm")


def upload_block(cfg: Config, layer: Dict[str, np.ndarray],
                 device: torch.device) -> Dict[str, torch.Tensor]:
    """Host arrays of one layer (``k_nope, v`` and the block weights) -> device tensors;
    ``k_cache``/``v_cache`` get room for the query rows after the context."""
    dt = layer_cfg(cfg).torch_dtype
    names = ("k_nope",) + BLOCK_WEIGHTS + tuple(v for v in VARIANT_WEIGHTS if v in layer)
    out = {name: torch.from_numpy(np.ascontiguousarray(layer[name])).to(dt).to(device)
           for name in names}
    n, qn = cfg.n_ctx, cfg.n_query
    v_cache = torch.zeros((n + qn, cfg.n_kv_heads, cfg.head_dim), dtype=dt, device=device)
    v_cache[:n] = torch.from_numpy(np.ascontiguousarray(layer["v"])).to(dt).to(device)
    out["v_cache"] = v_cache
    out["k_cache"] = torch.zeros_like(v_cache)
    return out


class CarriedRows:
    """Work buffers and call sequence for one configuration and MLP width."""

    def __init__(self, cfg: Config, inter: int, eps: float, device: torch.device,
                 k: Optional[int] = None, fuse_stage1: Optional[bool] = None):
        self.cfg, self.inter, self.eps, self.device = cfg, int(inter), float(eps), device
        self.lc = layer_cfg(cfg)
        n, qn = cfg.n_ctx, cfg.n_query
        # Stage I with one key stream less: the query rows' attention emits the
        # normaliser over the context keys and the score only sums the columns.
        # None = whenever the library has it for this geometry, but for the last scoring layer
        # of a whole run, whose attention nobody reads; True = there too
        ctx_ws = api.pkv_sparse_row_attn_ctx_lse_workspace_bytes(self.lc, n + qn, n, qn)
        self.fuse_stage1 = ctx_ws > 0 if fuse_stage1 is None else bool(fuse_stage1)
        self._fuse_last = bool(fuse_stage1)
        if self.fuse_stage1 and ctx_ws == 0:
            raise ValueError("fused Stage I is not available for this geometry")
        self.n, self.qn = n, qn
        self.k = select_count(cfg.ratio, n) if k is None else int(k)
        self.m = self.k + qn
        dt = self.lc.torch_dtype
        hq, hkv, d, hid = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.hidden
        i32 = dict(dtype=torch.int32, device=device)
        new = lambda *shape: torch.empty(shape, dtype=dt, device=device)  # noqa: E731
        self.q_rows = torch.arange(n, n + qn, **i32)
        self.rows = torch.empty(self.m, **i32)          # T_p ++ query rows
        self.rows[self.k:] = self.q_rows
        self.score = torch.zeros(n, dtype=torch.float32, device=device)
        self.lse_ctx = torch.empty((qn, hq), dtype=torch.float32, device=device)
        rows_max = max(self.m, qn)
        self.h = new(rows_max, hid)                     # carried hidden states
        self.x = new(rows_max, hid)                     # normalised rows
        self.q = new(rows_max, hq, d)
        self.attn = new(rows_max, hq, d)
        self.g = new(rows_max, self.inter)
        tdt = dt
        ws_bytes = 256
        for rows in (self.m, qn):
            ws_bytes = max(
                ws_bytes,
                api.pkv_workspace_bytes(api.CALL_SPARSE_ROW_ATTN, self.lc, n + qn, rows),
                api.pkv_workspace_bytes(api.CALL_GATHER_QKV_PROJ, self.lc, 0, rows),
                api.pkv_glue_workspace_bytes(tdt, rows, hq * d, hid),
                api.pkv_glue_workspace_bytes(tdt, rows, hid, self.inter),
                api.pkv_glue_workspace_bytes(tdt, rows, self.inter, hid))
        ws_bytes = max(ws_bytes, api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, self.lc, n, qn),
                       api.pkv_workspace_bytes(api.CALL_TOPK_SELECT, self.lc, n, 0), ctx_ws)
        self.ws = torch.empty(ws_bytes, dtype=torch.uint8, device=device)

    # one decoder layer for the first ``cnt`` rows of the buffers, at positions ``rows``;
    # caches_only: its normalisation and K/V projection, nothing of the rows themselves;
    # scores_only: up to the scores; chunks = (rows of the caches, chunk length): the rows are
    # all of the caches, in chunks that attend within themselves, ``rows`` counting inside them
    def _layer(self, L: Dict[str, torch.Tensor], rows: torch.Tensor, cnt: int,
               score: Optional[bool], caches_only: bool = False,
               scores_only: bool = False, chunks=None,
               ws: Optional[torch.Tensor] = None) -> None:
        # K and V go straight to their cache rows.  The score of Stage I reads only the context
        # rows of the key cache, which the query rows' own keys (stored behind the context) do
        # not touch.
        fused = score is not None and self.fuse_stage1 and chunks is None
        api.pkv_layer_rows(
            self.lc, self.h, self.x, self.q, self.attn, self.g, cnt, L, VARIANT_WEIGHTS,
            L["k_cache"], L["v_cache"], rows, rows if chunks is None else chunks[0], self.eps,
            self.ws if ws is None else ws, score=None if score is None else self.score,
            lse_ctx=self.lse_ctx if fused else None, n_ctx=self.n, accumulate=bool(score),
            chunk_len=0 if chunks is None else chunks[1],
            stop=api.LAYER_TO_CACHES if caches_only else
            api.LAYER_TO_SCORES if scores_only else api.LAYER_WHOLE)

    # the last scoring layer where only its scores are wanted: queries and both passes of the
    # score, which cost less than the attention that would spare one of them
    def _score_only(self, L: Dict[str, torch.Tensor], accumulate: bool) -> None:
        qn = self.qn
        api.pkv_rmsnorm_rows(self.h[:qn], None, L["w_in"], self.eps, self.x[:qn])
        api.pkv_gather_qkv_proj_ex(self.lc, self.x[:qn], None, self.q_rows, L["wq"], None, None,
                                   self.q[:qn], None, None, ws=self.ws, norm_eps=self.eps,
                                   **{v: L[v] for v in VARIANT_WEIGHTS if v in L})
        api.pkv_query_score(self.lc, self.q[:qn], L["k_cache"][:self.n], self.score,
                            accumulate=accumulate, ws=self.ws)

    def stage1(self, embed: torch.Tensor, layers: List[Dict[str, torch.Tensor]],
               n_score_layers: Optional[int] = None) -> None:
        """Restores every layer's context keys, scores with the query rows over the first
        ``n_score_layers`` layers and writes the selection into ``self.rows[:k]``.  The query
        rows' hidden states after those layers stay in ``self.h``, their K/V in the caches."""
        self._stage1(embed, layers, n_score_layers, keep_rows=True)

    # keep_rows=False: Stage II follows, which gathers the query rows anew and replaces their
    # cache rows in every layer - the last scoring layer then stops at its scores
    def _stage1(self, embed: torch.Tensor, layers: List[Dict[str, torch.Tensor]],
                n_score_layers: Optional[int], keep_rows: bool) -> None:
        ls = self.cfg.n_score_layers if n_score_layers is None else n_score_layers
        last = min(ls, len(layers)) - 1
        api.pkv_gather_rows(embed, self.q_rows, self.h[:self.qn])
        together = restore_together(self.lc, layers, self.n)
        for li, L in enumerate(layers):
            if not together:
                api.pkv_rope_restore(self.lc, L["k_nope"], L["k_cache"][:self.n], None, 0)
            if li == last and not keep_rows and self._fuse_last:
                self._layer(L, self.q_rows, self.qn, score=li > 0, scores_only=True)
            elif li == last and not keep_rows:
                self._score_only(L, accumulate=li > 0)
            elif li < ls:
                self._layer(L, self.q_rows, self.qn, score=li > 0)
        api.pkv_topk_select(self.score, self.k, self.rows, ws=self.ws)

    def stage2(self, embed: torch.Tensor, layers: List[Dict[str, torch.Tensor]]) -> torch.Tensor:
        """The rows ``self.rows`` through every layer; returns their final hidden states
        (a view of the work buffer).  Caches are updated in place."""
        self._stage2(embed, layers)
        return self.h[:self.m]

    def _stage2(self, embed: torch.Tensor, layers: List[Dict[str, torch.Tensor]]) -> None:
        api.pkv_gather_rows(embed, self.rows, self.h[:self.m])
        for L in layers:
            self._layer(L, self.rows, self.m, score=None)

    def run(self, embed, layers, n_score_layers: Optional[int] = None) -> torch.Tensor:
        self._stage1(embed, layers, n_score_layers, keep_rows=False)
        return self.stage2(embed, layers)
