"""The zero features of blocks that blend nothing are written by the selection up to
256 channels (in rows of more than 8 vectors, K <= 16) and by the gather otherwise: every element is written (the image starts as
NaN) and equals the fused render's, on both sides of that line."""
from __future__ import annotations

import pytest
import torch

from paper_2604_10951_amd import raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,K,dtype", [
    (32, 8, "f32"), (36, 8, "f32"), (64, 16, "bf16"), (72, 16, "bf16"), (256, 8, "f32"), (257, 8, "f32"),
    (260, 16, "f32"), (260, 20, "f32"), (1024, 3, "f32"), (256, 8, "bf16"), (264, 8, "bf16"), (520, 16, "bf16")])
def test_wide_images(C, K, dtype):
    print(f"[case] zero blocks, wide C={C} K={K} {dtype}", flush=True)
    scene = scenes.uniform_scene(60, seed=4, scale_range=(0.01, 0.04), feat_channels=C - 3)
    cam = scenes.centred_camera(101, 77)
    tens = raster.scene_tensors(scene, "cuda", dtype)
    rast = raster.Rasterizer(cam, tile=8, topk=K, schedule="split", feat_dtype=dtype, device="cuda")
    rast.render(*tens)
    out = rast.alloc_out(C)
    out["feat"].fill_(float("nan"))
    rast.render_forward(tens[4], out=out)
    full = raster.Rasterizer(cam, tile=8, topk=K, schedule="grid", feat_dtype=dtype, device="cuda").render(*tens)
    torch.cuda.synchronize()
    assert bool((out["n"] == 0).any()) and bool((out["n"] > 0).any())
    assert torch.equal(out["feat"], full.feat) and torch.equal(out["n"], full.n)
