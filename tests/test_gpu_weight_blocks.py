"""Top-K by weight: which blocks take a workgroup each depends on how many tile lists
are long (all of them if few are, the longest, or none).  The image depends neither
on that nor on the binning tile, so renders of one scene with different tiles, whose
lists differ in length, must agree bit for bit in every regime."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2604_10951_amd import raster, scenes

pytestmark = pytest.mark.gpu


def _lists(fr, tile):
    n = np.repeat((fr.ranges[:, 1] - fr.ranges[:, 0]).cpu().numpy(), (tile // 8) ** 2)
    return int((n > 48).sum()), int((n > 256).sum())


@pytest.mark.parametrize("n,W,H,K,want", [
    (2000, 128, 96, 8, ["all", "all", "all"]),             # few blocks
    (60000, 640, 480, 8, ["all", "longest", "longest"]),
    (300000, 1280, 720, 8, ["longest", "longest", "none"]),
    (100000, 640, 480, 16, ["all", "longest", "longest"]),
])
def test_regimes_agree(n, W, H, K, want):
    print(f"[case] by-weight blocks n={n} {W}x{H} K={K}", flush=True)
    scene = scenes.clustered_scene(n, 8, seed=1) if n > 2000 else scenes.uniform_scene(n, seed=2, feat_channels=5)
    cam = scenes.centred_camera(W, H)
    tens = raster.scene_tensors(scene, "cuda")
    got, regimes = [], []
    for tile in (8, 16, 32):
        fr = raster.Rasterizer(cam, tile=tile, topk=K, topk_mode="weight", device="cuda").render(*tens, want_idx=True)
        torch.cuda.synchronize()
        long, longest = _lists(fr, tile)
        regimes.append("all" if long <= 1024 else "longest" if longest <= 2560 else "none")
        got.append(fr)
    assert regimes == want, regimes
    for fr in got[1:]:
        for name in ("feat", "T", "n", "idx"):
            assert torch.equal(getattr(fr, name), getattr(got[0], name)), name
