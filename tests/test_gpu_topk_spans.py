"""The one-workgroup top-k on vectors whose keys span nothing, two values, all finite floats or
everything from -inf to +inf, whose threshold falls into one crowded bin, and of lengths around the
edges of its register layouts: indices bit-exact against the oracle (no tolerance)."""

import numpy as np
import pytest

from oracle import pkv_oracle as O
from tests.test_gpu_kernels import run_topk

pytestmark = pytest.mark.gpu


def vector(kind, n, g):
    if kind == "equal":
        return np.full(n, 0.25, np.float32)
    if kind == "two":
        return np.where(g.random(n) < 0.3, np.float32(1.0), np.float32(np.nextafter(1.0, 2.0, dtype=np.float32)))
    if kind == "infinite":
        s = g.standard_normal(n).astype(np.float32)
        s[::5], s[1::7] = -np.inf, np.inf
        return s
    if kind == "crowded":       # one far outlier at each end, the rest within a few thousand floats
        s = np.float32(1.0) + g.integers(0, 4000, n).astype(np.float32) * np.float32(2.0 ** -23)
        s[0], s[-1] = -3.0e38, 3.0e38
        return s
    bits = g.integers(0, 2 ** 32, n, dtype=np.uint64).astype(np.uint32)   # every finite float
    s = bits.view(np.float32).copy()
    s[~np.isfinite(s)] = 0.0
    return s


@pytest.mark.parametrize("kind", ["equal", "two", "infinite", "crowded", "floats"])
@pytest.mark.parametrize("n", [1, 257, 4099, 8192, 8193, 16384, 32767, 32768, 65536])
def test_spans(gpu_device, kind, n):
    s = vector(kind, n, np.random.default_rng(n))
    for k in sorted({1, max(1, n // 5), max(1, n - 1), n}):
        assert np.array_equal(run_topk(s, k, gpu_device), O.topk_select(s, k)), k
