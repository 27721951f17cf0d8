"""GPU parity of the attention whose key ranges are queued by weight: rows spread over the keys, all at
their end and in any order (the list is then not by weight, but still one of every job), with
tiles that the last row does not fill and caches that end inside a tile."""

import numpy as np
import pytest

from paper_2602_02579_amd import api
from tests.test_gpu_attn_short_ranges import check, planned_ranges
from tests.test_gpu_kernels import lcfg, rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["spread", "end", "any"])
@pytest.mark.parametrize("m,n_keys,hq,hkv,ranges", [
    (775, 5000, 32, 8, 4),        # 13 tiles x 4 ranges x 8 heads = 416 jobs
    (640, 8001, 40, 8, 4),        # 250 of 256 columns; the cache ends in a tile of 64 keys
    (1030, 10001, 16, 16, 5)])    # heads of their own, 400 jobs
def test_ranges_by_weight(gpu_device, m, n_keys, hq, hkv, ranges, order):
    cfg = lcfg("bf16", hq, hkv, 128)
    assert planned_ranges(cfg, n_keys, m) == ranges
    assert api.pkv_sparse_row_attn_kernel(cfg, n_keys, m) == api.ATTN_QUEUE_BY_WEIGHT
    q, kc, vc = (rnd(s, shape, "bf16") for s, shape in
                 ((1, (m, hq, 128)), (2, (n_keys, hkv, 128)), (3, (n_keys, hkv, 128))))
    if order == "end":
        pos = np.arange(n_keys - m, n_keys)
    else:
        pos = np.random.default_rng(m).choice(n_keys, m, replace=False)
        pos[:2] = [0, n_keys - 1]
        if order == "spread":
            pos.sort()
    check(gpu_device, hq, hkv, q, kc, vc, pos.astype(np.int32))
