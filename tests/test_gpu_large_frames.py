"""Frames of more than 2^23 render blocks, whose block launches take several rows of
workgroups: a small view packed behind a view of 32,767 x 16,640 pixels must give
the outputs, counts and gradients that it gives alone."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2604_10951_amd import raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,schedule", [(0, "grid"), (2, "grid"), (1, "split")])
def test_view_behind_a_very_large_one(K, schedule):
    print(f"[case] large frame K={K} {schedule}", flush=True)
    if torch.cuda.get_device_properties(0).total_memory < 64 << 30:
        pytest.skip("needs 64 GB of GPU memory")
    scene = scenes.uniform_scene(300, seed=3, rgb=1, feat_channels=0, scale_range=(0.02, 0.08))
    tens = raster.scene_tensors(scene, "cuda")
    small = scenes.centred_camera(93, 71)
    away = scenes.Camera(32767, 16640, 20000.0, 20000.0, 16000.0, 8000.0, R=np.diag([1.0, -1.0, -1.0]))
    rast = raster.Rasterizer([away, small], tile=32, topk=K, schedule=schedule, device="cuda")
    assert rast.total_tiles * 16 > 1 << 23
    fr = rast.render(*tens, want_last=True)
    alone = raster.Rasterizer(small, tile=32, topk=K, schedule=schedule, device="cuda")
    want = alone.render(*tens, want_last=True)
    torch.cuda.synchronize()
    first = away.width * away.height
    for name in ("feat", "T", "n"):
        a, b = getattr(fr, name), getattr(want, name)
        assert torch.equal(a[first:], b), name
    assert int(fr.n[:first].max()) == 0 and float(fr.feat[:first].abs().max()) == 0.0
    assert int(want.n.sum()) > 100
    if K > 0:
        return
    grad = torch.zeros_like(fr.feat)
    g = torch.randn(want.feat.shape, generator=torch.Generator().manual_seed(1)).cuda()
    grad[first:] = g
    got, ref = rast.render_backward(*tens, fr, grad), alone.render_backward(*tens, want, g)
    torch.cuda.synchronize()
    # a surfel's blocks are summed by float atomics in any order (a few partial sums,
    # 2^-24 each), which the projection's chain can amplify; a block left out or taken
    # twice changes the sums by their own size
    for name in ref:
        scale = float(ref[name].abs().max())
        assert scale > 0 and float((got[name] - ref[name]).abs().max()) <= 1e-3 * scale, name
