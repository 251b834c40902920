"""The persistent schedule's work queue: frames of more render blocks than any
device holds at once (eight workgroups per CU), so that workgroups take several
blocks each and reuse their LDS from one to the next.  Every form of the block
kernel must give the plain grid's outputs, bit for bit, also as a replayed graph
whose tickets start anew."""
from __future__ import annotations

import pytest
import torch

from paper_2604_10951_amd import raster, scenes

pytestmark = pytest.mark.gpu

W, H, N = 1289, 727, 60000   # more surfels than 8x8 blocks; remainders on both sides


def _assert_queued(rast, n):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tile = int(rast.opts.tile)
    blocks = rast.total_tiles * (tile // 8) ** 2
    assert blocks > 8 * cus and n >= blocks, (blocks, cus)


def _tensors(C, dtype="f32"):
    return raster.scene_tensors(scenes.clustered_scene(N, C, seed=2), "cuda", dtype)


@pytest.mark.parametrize("tile,batch,K,C,dtype,extra", [
    (8, 32, 0, 5, "f32", {}), (8, 16, 0, 16, "f32", {}), (16, 32, 0, 33, "f32", {}), (16, 16, 3, 8, "f32", {}),
    (32, 32, 0, 12, "f32", {}), (32, 16, 0, 72, "bf16", {}), (8, 32, 4, 100, "f32", {}),
    (8, 32, 0, 3, "f32", {"geo": True}), (16, 32, 0, 8, "f32", {"geo": True}), (32, 32, 2, 4, "bf16", {"geo": True}),
    (16, 32, 0, 8, "f32", {"lowpass": True})])
def test_queue_matches_the_grid(tile, batch, K, C, dtype, extra):
    print(f"[case] queue tile={tile} batch={batch} K={K} C={C} {dtype} {extra}", flush=True)
    cam, tens = scenes.centred_camera(W, H), _tensors(C, dtype)
    geo, low = extra.get("geo", False), extra.get("lowpass", False)
    got = []
    for schedule in ("grid", "persistent"):
        rast = raster.Rasterizer(cam, tile=tile, batch=batch, topk=K, feat_dtype=dtype, schedule=schedule, lowpass=low,
                                 device="cuda")
        _assert_queued(rast, N)
        for _ in range(2):   # (the second frame finds the first one's tickets)
            fr = rast.render(*tens, want_last=True, want_idx=K > 0, want_depth=geo, want_normal=geo)
        torch.cuda.synchronize()
        got.append(fr)
    for name in ("feat", "T", "n", "last", "idx", "depth", "normal"):
        x, y = getattr(got[0], name), getattr(got[1], name)
        assert (x is None and y is None) or torch.equal(x, y), name
    assert int((got[0].n > 0).sum()) > 1000


def test_queue_in_a_replayed_graph():
    print("[case] queue in a graph", flush=True)
    cam, tens = scenes.centred_camera(W, H), _tensors(6)
    rast = raster.Rasterizer(cam, tile=16, schedule="persistent", device="cuda")
    _assert_queued(rast, N)
    graph = raster.FrameGraph(rast, tens)
    ref = raster.Rasterizer(cam, tile=16, schedule="grid", device="cuda")
    for k in range(4):
        tens[3].mul_(0.9)                       # new inputs between the replays
        want = ref.render(*tens)
        out = graph.replay()
        torch.cuda.synchronize()
        assert graph.pairs_fit()
        for name in ("feat", "T", "n"):
            assert torch.equal(out[name], getattr(want, name)), (k, name)
