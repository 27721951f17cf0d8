"""GPU parity of the attention whose jobs are 128 columns with the keys shared by two groups of waves
(contexts of a few thousand keys): row limits at the edges of its 32-key blocks and of the pairs of
them, caches that end inside a block, groups whose rows do not fill the columns, rows in any order, rows
that see a single key, scores that keep growing (the second attempt), and the counts of jobs and keys
where the launch goes to it."""

import numpy as np
import pytest

from paper_2602_02579_amd import synth
from tests.test_gpu_attn_short_ranges import check
from tests.test_gpu_kernels import rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("growing", [False, True])
@pytest.mark.parametrize("m,n_keys,hq,hkv,order", [
    (200, 1120, 32, 8, "sorted"),      # 56 jobs: as few as 1120 keys take
    (200, 1121, 32, 8, "sorted"),      # a key too many
    (1030, 1030, 40, 8, "sorted"),     # 336 jobs, 125 of 128 columns
    (1024, 1040, 32, 8, "sorted"),     # 256 jobs
    (700, 1503, 35, 5, "any"),         # groups of seven heads, cache ends inside a block
    (400, 1217, 16, 16, "any"),        # groups of one: 128 rows a job
    (100, 1089, 64, 8, "end")])
def test_pairs(gpu_device, m, n_keys, hq, hkv, order, growing):
    q, vc = rnd(1, (m, hq, 128), "bf16"), rnd(3, (n_keys, hkv, 128), "bf16")
    kc = rnd(2, (n_keys, hkv, 128), "bf16")
    if growing:   # up to ~60 nats between the first and the last key
        kc = synth.to_storage(kc * np.linspace(0.05, 5.0, n_keys, dtype=np.float32)[:, None, None],
                              "bf16")
    gen = np.random.default_rng(m)
    if order == "end":
        pos = np.arange(n_keys - m, n_keys)
    else:
        pos = gen.choice(n_keys, m, replace=False)
        edges = [0, 1, 30, 31, 32, 33, 62, 63, 64, 65, 95, 96, 127, 128, 129, n_keys - 1]
        pos[:len(edges)] = edges
        if order == "sorted":
            pos.sort()
    check(gpu_device, hq, hkv, q, kc, vc, pos.astype(np.int32))
