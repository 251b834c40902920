"""Blocks that blend nothing: the selection pass writes their zero features and
the gather leaves them alone.  The output buffer starts out as NaN, so a block
written by neither shows; ragged images, both gathers, K beyond the compact
lists and empty scenes."""
from __future__ import annotations

import pytest
import torch

from paper_2604_10951_amd import raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C_extra,K,tile,n", [(13, 8, 8, 40), (14, 8, 16, 40), (297, 3, 32, 40), (61, 24, 8, 40),
                                              (125, 16, 8, 0)])
def test_blocks_without_contributors_are_zero(C_extra, K, tile, n):
    print(f"[case] zero blocks C={C_extra + 3} K={K} tile={tile} n={n}", flush=True)
    scene = scenes.uniform_scene(max(n, 1), seed=3, feat_channels=C_extra)
    if n == 0:
        scene.opacity[:] = 1e-4   # every surfel is culled
    tens = raster.scene_tensors(scene, "cuda")
    cams = [scenes.centred_camera(101, 77), scenes.centred_camera(67, 90)]
    rast = raster.Rasterizer(cams, tile=tile, topk=K, schedule="split", device="cuda")
    rast.render(*tens)
    out = rast.alloc_out(scene.channels)
    out["feat"].fill_(float("nan"))
    rast.render_nosync(*tens, out)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out["feat"]).all())
    empty = out["n"] == 0
    assert bool(empty.any()) and (n == 0) == bool(empty.all())
    assert int(torch.count_nonzero(out["feat"][empty])) == 0
    full = raster.Rasterizer(cams, tile=8, topk=K, schedule="grid", device="cuda").render(*tens)
    assert torch.equal(full.feat, out["feat"])


@pytest.mark.parametrize("K,n", [(8, 30000), (16, 30000), (3, 6000)])
def test_by_weight_long_lists(K, n):
    """By weight, blocks with long tile lists (here of a few hundred entries,
    walked by two waves): transmittance and, where K covers every contributor,
    features of the full blend; n = min(K, contributors)."""
    print(f"[case] weight long lists K={K} n={n}", flush=True)
    scene = scenes.uniform_scene(n, seed=8, scale_range=(0.004, 0.02), feat_channels=13)
    tens = raster.scene_tensors(scene, "cuda")
    cam = scenes.centred_camera(90, 70)
    fr = raster.Rasterizer(cam, tile=8, topk=K, topk_mode="weight", device="cuda").render(*tens, want_idx=True)
    full = raster.Rasterizer(cam, tile=8, topk=0, device="cuda").render(*tens)
    torch.cuda.synchronize()
    lens = fr.ranges[:, 1] - fr.ranges[:, 0]
    assert int(lens.max()) > 48
    assert torch.equal(fr.n, full.n.clamp(max=K)) and torch.equal(fr.T, full.T)
    all_in = full.n <= K
    assert torch.equal(fr.feat[all_in], full.feat[all_in])
    assert bool(((fr.idx >= 0).sum(1) == fr.n).all())
    assert bool((fr.idx[~all_in] >= 0).all())
