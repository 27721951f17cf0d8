"""GPU parity of the attention over caches of up to 1024 keys with at most one job of 128 columns
per compute unit: one key, key counts around the 64-key tiles and the 128-key pairs of them,
groups whose rows do not fill the columns, rows that see a single key, scores that keep growing
along the keys (every tile raises the maximum), and the launches just above both limits."""

import numpy as np
import pytest

from paper_2602_02579_amd import synth
from tests.test_gpu_attn_short_ranges import check
from tests.test_gpu_kernels import rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("growing", [False, True])
@pytest.mark.parametrize("m,n_keys,hq,hkv", [
    (1, 1, 2, 2), (33, 64, 8, 2), (64, 65, 8, 2), (65, 127, 8, 2), (256, 256, 8, 2),
    (129, 129, 10, 2), (100, 193, 14, 2), (512, 512, 32, 8), (700, 1024, 10, 2), (40, 1024, 32, 2),
    (1025, 1025, 8, 2),          # one key too many
    (1024, 1024, 32, 8),         # 256 jobs
    (1023, 1023, 36, 9)])        # more than 256
def test_short_caches(gpu_device, m, n_keys, hq, hkv, growing):
    q, vc = rnd(1, (m, hq, 128), "bf16"), rnd(3, (n_keys, hkv, 128), "bf16")
    kc = rnd(2, (n_keys, hkv, 128), "bf16")
    if growing:   # up to ~60 nats between the first and the last key
        kc = synth.to_storage(kc * np.linspace(0.05, 5.0, n_keys, dtype=np.float32)[:, None, None], "bf16")
    pos = np.arange(n_keys - m, n_keys, dtype=np.int32) if m <= n_keys else None
    if m > 2:
        pos[:2] = (0, 1) if pos[2] >= 2 else pos[:2]
    check(gpu_device, hq, hkv, q, kc, vc, pos)
