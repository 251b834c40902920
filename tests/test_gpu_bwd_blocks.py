"""Full-blend backward over long and filtered lists: tiles of 32x32 and 16x16
pixels queue the entries that meet a block (lists of several thousand entries,
walked back to front in many refills), 8x8 tiles walk them directly; channel
counts at the edges of the per-thread channel groups (16, 32, 48, 64, 128)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2604_10951_amd import scenes
from tests.test_gpu_backward import _check, _gpu_grads, _upstream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,tile,C_extra,dtype", [
    (9000, 32, 13, "f32"), (9000, 16, 14, "f32"), (9000, 8, 30, "f32"), (300, 32, 45, "f32"), (300, 8, 46, "f32"),
    (300, 16, 62, "f32"), (300, 16, 125, "f32"), (300, 8, 61, "bf16"),
])
def test_full_blend_backward_blocks(n, tile, C_extra, dtype):
    print(f"[case] bwd blocks n={n} tile={tile} C={C_extra + 3} {dtype}", flush=True)
    scene = scenes.uniform_scene(n, seed=17, feat_channels=C_extra)
    if dtype == "bf16":   # the oracle differentiates the stored (rounded) features
        import torch
        scene.feats[:] = torch.from_numpy(scene.feats).bfloat16().float().numpy()
    cam = scenes.centred_camera(77, 61)
    g = _upstream(scene, cam, 0, seed=2)
    gpu = _gpu_grads(scene, cam, g, tile=tile, topk=0, feat_dtype=dtype)
    ref = oracle.render_grad(scene.means, scene.scales, scene.quats, scene.opacity, scene.feats, cam, g, K=0,
                             with_abs=True)
    assert np.abs(gpu["feats"]).sum() > 0
    _check(gpu, ref, f"bwd n={n} tile={tile} C={scene.channels} {dtype}")


@pytest.mark.parametrize("C,K,dtype", [(16, 8, "f32"), (20, 3, "f32"), (48, 16, "f32"), (64, 8, "f32"), (132, 8, "f32"),
                                       (256, 4, "f32"), (64, 8, "bf16"), (264, 5, "bf16")])
def test_topk_backward_channel_groups(C, K, dtype):
    """Top-K backward at the edges of its channel groups (16 threads per row
    slot up to 128 channels, 32 up to 256, 64 beyond)."""
    print(f"[case] topk bwd C={C} K={K} {dtype}", flush=True)
    scene = scenes.uniform_scene(600, seed=23, feat_channels=C - 3)
    if dtype == "bf16":
        import torch
        scene.feats[:] = torch.from_numpy(scene.feats).bfloat16().float().numpy()
    cam = scenes.centred_camera(61, 50)
    g = _upstream(scene, cam, K, seed=4)
    gpu = _gpu_grads(scene, cam, g, tile=8, topk=K, feat_dtype=dtype)
    ref = oracle.render_grad(scene.means, scene.scales, scene.quats, scene.opacity, scene.feats, cam, g, K=K,
                             with_abs=True)
    assert np.abs(gpu["feats"]).sum() > 0
    _check(gpu, ref, f"topk bwd C={C} K={K} {dtype}")
