"""render() enqueues the whole frame before it reads the pair count back: a
frame that does not fit its pair buffers is taken again with larger ones, on
any stream, and equals the frame of a rasterizer that had room from the start."""
from __future__ import annotations

import pytest
import torch

from paper_2604_10951_amd import raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("topk,side_stream", [(0, False), (8, True)])
def test_frame_that_outgrows_its_pair_buffers(topk, side_stream):
    print(f"[case] capacity topk={topk} side_stream={side_stream}", flush=True)
    small, cam = scenes.parity_small()
    big = scenes.uniform_scene(small.n, seed=9, scale_range=(0.02, 0.2))   # many more pairs
    ref = raster.Rasterizer(cam, tile=8, topk=topk, device="cuda", pair_capacity=1 << 20)
    stream = torch.cuda.Stream() if side_stream else torch.cuda.current_stream()
    t_small, t_big = raster.scene_tensors(small, "cuda"), raster.scene_tensors(big, "cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        rast = raster.Rasterizer(cam, tile=8, topk=topk, device="cuda", pair_capacity=1024)
        for tens in (t_small, t_big, t_small):
            capacity = rast.capacity
            a = rast.render(*tens, want_last=True)
            b = ref.render(*tens, want_last=True)
            torch.cuda.synchronize()
            assert a.num_pairs == b.num_pairs == int(rast._bufs["num_pairs"].item())
            assert rast.capacity >= a.num_pairs and (rast.capacity > capacity) == (a.num_pairs > capacity)
            for name in ("feat", "T", "n", "last", "ranges"):
                assert torch.equal(getattr(a, name), getattr(b, name)), name
            P = a.num_pairs
            assert torch.equal(a.keys[:P], b.keys[:P]) and torch.equal(a.vals[:P], b.vals[:P])
    assert rast.capacity > 1024
