"""Host checks of the chunk producer, which run before any library call."""

import pytest
import torch

from paper_2602_02579_amd import diagnostics
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
