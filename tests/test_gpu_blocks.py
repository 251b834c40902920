"""Render blocks that see only a part of their tile's list (16x16 and 32x32
binning tiles): the entries are queued by their pixel boxes before the walk.
Images do not depend on the binning tile, so every output must be bit-identical
to the 8x8-tile render, which walks its lists unfiltered, and meet the oracle's
bars.  The dense scene's 32x32 tiles hold several thousand entries (many
refills, the queue wrapping round), the sparse one less than a batch."""
from __future__ import annotations

import pytest
import torch

import oracle
from paper_2604_10951_amd import raster, scenes
from tests.test_gpu_parity import check_image

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,tile,K,C_extra,geo,schedule", [
    (12000, 32, 0, 13, False, "persistent"),
    (12000, 16, 0, 14, False, "grid"),
    (12000, 32, 5, 61, False, "grid"),
    (12000, 8, 0, 45, False, "persistent"),   # C = 48: rows of 12 lanes
    (12000, 32, 0, 125, True, "persistent"),
    (150, 32, 0, 13, True, "grid"),
    (150, 16, 3, 14, False, "persistent"),
])
def test_larger_tiles_render_the_same_image(n, tile, K, C_extra, geo, schedule):
    print(f"[case] blocks n={n} tile={tile} K={K} C={C_extra + 3} geo={geo} {schedule}", flush=True)
    scene = scenes.uniform_scene(n, seed=31, feat_channels=C_extra)
    cam = scenes.centred_camera(101, 77)
    tens = raster.scene_tensors(scene, "cuda")
    got = []
    for t in (8, tile):
        rast = raster.Rasterizer(cam, tile=t, topk=K, schedule=schedule, device="cuda")
        fr = rast.render(*tens, want_last=True, want_idx=K > 0, want_depth=geo, want_normal=geo)
        torch.cuda.synchronize()
        if t > 8:
            longest = int((fr.ranges[:, 1] - fr.ranges[:, 0]).max())
            assert longest > 1024 if n > 1000 else longest < 300, longest
        got.append((fr, rast))
    a, b = got[0][0], got[1][0]
    for name in ("feat", "T", "n", "idx", "depth", "normal"):
        x, y = getattr(a, name), getattr(b, name)
        assert (x is None and y is None) or torch.equal(x, y), name
    # the last blended entry is the same record, at each list's own position
    on = a.last >= 0
    assert torch.equal(on, b.last >= 0)
    assert torch.equal(a.vals[a.last[on].long()], b.vals[b.last[on].long()])
    ref = oracle.render_scene(scene, cam, K=K, kcap=max(K, 1))
    check_image(b, ref, got[1][1], 0, scene.channels, K, f"blocks tile {tile}")
