"""Scratch of the fp32 query score: with many columns (query tokens x heads) a float for each, which
is what lets pkv_query_score_static, whose scratch is fixed, take 4M of them."""

import ctypes
import os

import pytest

from paper_2602_02579_amd import api


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (32, 8, 128), (8, 1, 32)])
@pytest.mark.parametrize("n", [1, 100, 32768, 1 << 20])
def test_many_columns_need_a_float_each(hq, hkv, d, n):
    if not os.path.exists(api.library_path()):
        pytest.skip("libpkv.so not built")
    cfg = api.LayerCfg(hq, hkv, d, 256, 1e4, "f32")
    for cols in (8192 + 2 * hq, 1 << 20, 1 << 22):
        nq = cols // hq
        assert api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, cfg, n, nq) == \
            (nq * hq * 4 + 255) // 256 * 256
    # few columns: a pair per split and column, 8192 pairs and a split more at most
    for nq in (1, 16, 200):
        if nq * hq <= 8192:
            assert api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, cfg, n, nq) <= 2 * 8192 * 8


def test_the_static_call_takes_as_many_columns_as_before():
    """It checks its scratch first, on the host; null pointers end the call behind that, or the
    missing device does."""
    if not os.path.exists(api.library_path()):
        pytest.skip("libpkv.so not built")
    lib = api.load_library()
    c = api.LayerCfg(32, 8, 128, 4096, 1e4, "f32")._c()
    need = api.pkv_workspace_bytes(api.CALL_QUERY_SCORE, api.LayerCfg(32, 8, 128, 4096, 1e4, "f32"),
                                   64, (1 << 22) // 32)
    assert need <= api.STATIC_SCRATCH_BYTES
    workspace_error = 4
    assert lib.pkv_query_score_static(ctypes.byref(c), None, None, None, (1 << 22) // 32, 64, 0.0, 0,
                                      None) != workspace_error
