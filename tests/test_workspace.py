"""The rasterizer's workspace follows its options: they can be changed between
frames, and every frame's kernels write as much scratch as the options ask for
(the Top-K lists grow with K)."""
from __future__ import annotations

import ctypes

import pytest

from paper_2604_10951_amd import raster, scenes


@pytest.mark.parametrize("before,after", [({"topk": 1}, {"topk": 16}), ({"topk": 0}, {"topk": 4, "schedule": 2})])
def test_workspace_grows_with_the_options(before, after):
    rast = raster.Rasterizer(scenes.centred_camera(64, 48), topk=before["topk"], device="cpu")
    rast._ensure(100, 4096)
    for name, value in after.items():
        setattr(rast.opts, name, value)
    rast._ensure(100, 4096)
    need = rast.lib.fs_workspace_bytes(100, 1, rast.total_tiles, rast.capacity, ctypes.byref(rast.opts))
    assert rast._bufs["ws"].numel() >= need
