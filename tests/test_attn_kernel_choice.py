"""Which attention kernel a call runs is a host function of its sizes: both sides of every edge of the
rules, and what the call refuses."""

import os

import pytest

from paper_2602_02579_amd import api

pytestmark = pytest.mark.skipif(not os.path.exists(api.library_path()), reason="libpkv.so not built")


@pytest.fixture(autouse=True)
def choice_by_size(monkeypatch):
    monkeypatch.delenv("PKV_ATTN_VT", raising=False)
    monkeypatch.delenv("PKV_ATTN_RANGES", raising=False)


def kernel(hq, hkv, n_keys, m, d=128, dtype="bf16"):
    return api.pkv_sparse_row_attn_kernel(api.LayerCfg(hq, hkv, d, 256, 1e4, dtype), n_keys, m)


@pytest.mark.parametrize("hq,hkv,n_keys,m,pairs", [
    # up to one job per CU: twenty keys a job
    (32, 8, 1120, 200, True), (32, 8, 1121, 200, False),
    (32, 8, 5120, 1024, True), (32, 8, 5121, 1024, False), (32, 8, 5121, 1025, True),
    # up to two and a half jobs per CU, up to 12k keys
    (32, 8, 4000, 2560, True), (32, 8, 4000, 2561, False),
    (32, 8, 12288, 2000, True), (32, 8, 12289, 2000, False),
    # a third job per CU, where tiles of twice the columns are one per CU, and one tile more
    (40, 8, 4000, 1600, True), (40, 8, 4000, 1601, False), (40, 8, 4000, 1632, False),
    (40, 8, 4000, 1633, True),
    # groups that leave more than a twentieth of the columns empty: one job per CU at most
    (96, 8, 4000, 320, True), (96, 8, 4000, 321, False), (128, 8, 4000, 257, True),
    # large groups over few keys: one and a half
    (64, 8, 1535, 768, True), (64, 8, 1535, 769, False), (64, 8, 1536, 769, True),
    (40, 8, 1535, 1500, True)])
def test_where_the_keys_are_shared_in_pairs(hq, hkv, n_keys, m, pairs):
    assert (kernel(hq, hkv, n_keys, m) == api.ATTN_PAIRS) == pairs


def test_the_others():
    assert kernel(32, 8, 1024, 1000) == api.ATTN_SHORT
    assert kernel(32, 8, 32768, 64) == api.ATTN_ONE_JOB
    assert kernel(32, 8, 32768, 6681) == api.ATTN_QUEUE
    assert kernel(32, 8, 32900, 883) == api.ATTN_QUEUE_BY_WEIGHT
    assert kernel(28, 4, 32900, 1700) == api.ATTN_QUEUE          # fewer kv heads than XCDs
    assert kernel(8, 2, 1000, 100, d=64) == api.ATTN_TILES_64
    assert kernel(64, 2, 1000, 100) == api.ATTN_GENERIC          # groups of more than 16 heads
    assert kernel(8, 2, 1000, 100, d=64, dtype="f32") == api.ATTN_F32
    assert kernel(8, 2, 1000, 100, d=48, dtype="f32") == api.ATTN_GENERIC
    for n_keys, m in ((0, 5), (5, 0), (-1, 5), (5, -1), (1 << 24, 5), (1000, 1 << 27)):
        assert kernel(32, 8, n_keys, m) < 0
    assert kernel(32, 7, 1000, 100) < 0


def test_sources_of_the_values_that_leave_no_choice(monkeypatch):
    monkeypatch.setenv("PKV_ATTN_VT", "1")      # a transposed copy: neither short caches nor pairs
    assert kernel(32, 8, 4000, 1000) in (api.ATTN_ONE_JOB, api.ATTN_QUEUE)
    assert kernel(32, 8, 512, 512) in (api.ATTN_ONE_JOB, api.ATTN_QUEUE)
