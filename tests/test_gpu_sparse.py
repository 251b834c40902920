"""Frames with few surfels: most blocks blend nothing and are written as rows of
zeros, and with fewer surfels than blocks the work queue is left out.  Every output
element must be written (the buffers start as NaN), whatever the channel count and
the image's remainders, and the tiles must agree bit for bit."""
from __future__ import annotations

import pytest
import torch

import oracle
from paper_2604_10951_amd import raster, scenes
from tests.test_gpu_parity import check_image

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,C", [(40, 16), (40, 19), (40, 132), (1, 64), (1200, 48)])
@pytest.mark.parametrize("geo", [False, True])
def test_sparse_frames(n, C, geo):
    print(f"[case] sparse n={n} C={C} geo={geo}", flush=True)
    scene = scenes.uniform_scene(n, seed=n, scale_range=(0.005, 0.02), feat_channels=C - 3)
    cam = scenes.centred_camera(203, 149)
    tens = raster.scene_tensors(scene, "cuda")
    got = []
    for tile, schedule in ((8, "grid"), (8, "persistent"), (16, "persistent"), (32, "persistent")):
        rast = raster.Rasterizer(cam, tile=tile, schedule=schedule, device="cuda")
        fr = rast.render(*tens)
        out = rast.alloc_out(C, want_last=True, want_depth=geo, want_normal=geo)
        for k in ("feat", "T", "depth", "normal"):
            if out[k] is not None:
                out[k].fill_(float("nan"))
        out["n"].fill_(-7)
        rast.render_forward(tens[4], out=out)
        torch.cuda.synchronize()
        got.append(out)
        for k in ("feat", "T", "n"):
            assert torch.equal(out[k], getattr(fr, k)), k
    for out in got[1:]:
        for k in ("feat", "T", "n", "depth", "normal"):
            assert out[k] is None or torch.equal(out[k], got[0][k]), k
    assert (got[0]["n"] == 0).any() and torch.isfinite(got[0]["feat"]).all()
    check_image(fr, oracle.render_scene(scene, cam, K=0, kcap=1), rast, 0, C, 0, f"sparse {n}")
