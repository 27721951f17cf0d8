"""The keys of several layers restored by one call: the same bits as a call per layer, for more layers
than a launch holds, token counts that deal the heads out and that do not, in place and not, both
types, given positions and counted ones; and what the binding refuses."""

import pytest
import torch

from paper_2602_02579_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hkv,d", [("bf16", 8, 128), ("bf16", 3, 64), ("f32", 5, 32)])
@pytest.mark.parametrize("n,layers", [(1, 1), (37, 9), (700, 17), (5000, 3)])
@pytest.mark.parametrize("in_place", [False, True])
def test_layers(gpu_device, dtype, hkv, d, n, layers, in_place):
    cfg = api.LayerCfg(hkv, hkv, d, 64, 1e4, dtype)
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(n)
    src = [torch.randn((n, hkv, d), generator=gen, device=gpu_device).to(cfg.torch_dtype)
           for _ in range(layers)]
    pos = -torch.arange(n, dtype=torch.int32, device=gpu_device) if in_place else None
    want = [torch.empty_like(k) for k in src]
    for k, w in zip(src, want):
        api.pkv_rope_restore(cfg, k, w, pos, 11)
    out = src if in_place else [torch.zeros_like(k) for k in src]
    api.pkv_rope_restore_layers(cfg, src, out, pos, 11)
    for a, b in zip(out, want):
        assert torch.equal(a, b)


def test_lists_that_do_not_match_are_refused(gpu_device):
    cfg = api.LayerCfg(2, 2, 32, 64, 1e4, "f32")
    k = [torch.zeros((n, 2, 32), device=gpu_device) for n in (4, 4, 5)]
    with pytest.raises(ValueError):
        api.pkv_rope_restore_layers(cfg, k[:2], k[:1])
    with pytest.raises(ValueError):
        api.pkv_rope_restore_layers(cfg, k, k)
    api.pkv_rope_restore_layers(cfg, [], [])


def test_layers_that_share_memory_are_not_restored_together(gpu_device):
    room = torch.zeros((40, 2, 32), device=gpu_device)
    a, b, c = room[:10], room[10:20], room[5:15]
    assert api.caches_apart([], []) and api.caches_apart([a, b], [a, b])
    assert api.caches_apart([a, b], [room[20:30], room[30:]])
    for k_in, k_out in (([a, b], [c, room[20:30]]), ([a, b], [room[20:30], a]),
                        ([a, a], [b, room[20:30]]), ([a, b], [room[20:30], room[25:35]])):
        assert not api.caches_apart(k_in, k_out)
