"""CarriedRows(fuse_stage1=True): every scoring layer of a whole run takes its normaliser from
the query rows' attention, the last one (whose attention nobody reads) too.  stage1() alone runs
every layer in full, so the scores of both are the same calls on the same inputs: the same bits."""

import pytest
import torch

from paper_2602_02579_amd import model
from tests.test_gpu_model import CASES, EPS
from tests.test_gpu_run_without_dead_work import setup

pytestmark = pytest.mark.gpu

FUSED = [n for n, (cfg, _) in sorted(CASES.items())
         if cfg.dtype == "bf16" and cfg.head_dim == 128 and cfg.n_ctx % 64 == 0]


def test_there_are_geometries_that_fuse():
    assert FUSED


@pytest.mark.parametrize("n_score", [1, 2])
@pytest.mark.parametrize("name", FUSED)
def test_asked_for_fusion_reaches_the_last_scoring_layer(gpu_device, name, n_score):
    scores = []
    for whole in (True, False):
        cfg, inter, embed, layers = setup(name, gpu_device)
        cr = model.CarriedRows(cfg, inter, EPS, gpu_device, fuse_stage1=True)
        cr.lse_ctx.fill_(float("nan"))
        (cr.run if whole else cr.stage1)(embed, layers, n_score)
        assert cr.lse_ctx.isfinite().all()
        scores.append((cr.score.clone(), cr.rows.clone()))
    for a, b in zip(*scores):
        assert torch.equal(a, b)
