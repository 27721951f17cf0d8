"""pkv_workspace_bytes is a pure host function of any sizes: problems without tokens or rows, and
sizes beyond what the calls take, get an answer (in a process of their own: a division by zero
would end this one)."""

import os
import subprocess
import sys

import pytest

from paper_2602_02579_amd import api

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
from paper_2602_02579_amd import api
cfg = api.LayerCfg({hq}, {hkv}, {d}, 256, 1e4, "{dtype}")
for call in (api.CALL_QUERY_SCORE, api.CALL_TOPK_SELECT, api.CALL_GATHER_QKV_PROJ,
             api.CALL_SPARSE_ROW_ATTN):
    for n, m in ((0, 5), (5, 0), (0, 0), (1 << 32, 3000), (1 << 33, 1), (1 << 40, 5), (5, 3)):
        print(call, n, m, api.pkv_workspace_bytes(call, cfg, n, m))
"""


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128, 256])
def test_every_size_has_an_answer(dtype, d):
    if not os.path.exists(api.library_path()):
        pytest.skip("libpkv.so not built")
    run = subprocess.run([sys.executable, "-c", CODE.format(hq=4, hkv=2, d=d, dtype=dtype)],
                         cwd=ROOT, capture_output=True, text=True)
    assert run.returncode == 0, f"ended with {run.returncode} after {run.stdout.splitlines()[-1:]}"
    sizes = {tuple(map(int, line.split()[:3])): int(line.split()[3])
             for line in run.stdout.splitlines()}
    assert len(sizes) == 28
    assert sizes[api.CALL_QUERY_SCORE, 5, 0] == 0          # no query rows: nothing to keep
    # a call of any size has room for the normalisers of its columns
    assert sizes[api.CALL_QUERY_SCORE, 5, 3] >= 3 * 4 * 4
    assert sizes[api.CALL_QUERY_SCORE, 1 << 33, 1] >= 4 * 4
