"""render() enqueues a whole frame before it knows the frame's pair count, but not
where that is likely to be in vain: the first frame of its buffers, and frames whose
pairs come near the capacity, wait for the count before anything is sorted.  A frame
that outgrows its buffers all the same is taken again and comes out right.  Frames
make no events or pinned buffers of their own."""
from __future__ import annotations

import pytest
import torch

from paper_2604_10951_amd import raster, scenes

pytestmark = pytest.mark.gpu


class Calls:
    """The library, counting the calls of every entry point."""

    def __init__(self, lib):
        self.lib, self.count = lib, {}

    def __getattr__(self, name):
        fn = getattr(self.lib, name)

        def call(*args):
            self.count[name] = self.count.get(name, 0) + 1
            return fn(*args)
        return call


def _setup(capacity, **kw):
    scene = scenes.uniform_scene(3000, seed=6, feat_channels=13)
    rast = raster.Rasterizer(scenes.centred_camera(160, 120), pair_capacity=capacity, device="cuda", **kw)
    rast.lib = Calls(rast.lib)
    return rast, raster.scene_tensors(scene, "cuda")


def _same(a, b):
    for k in ("feat", "T", "n"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    assert a.num_pairs == b.num_pairs


def test_first_frame_that_outgrows_its_buffers_renders_once():
    print("[case] first frame outgrows", flush=True)
    rast, tens = _setup(64)
    fr = rast.render(*tens)
    assert fr.num_pairs > 64 and rast.capacity >= fr.num_pairs
    assert rast.lib.count["fs_render_forward"] == 1 and rast.lib.count["fs_bin"] == 2
    ref, _ = _setup(1 << 20)
    _same(fr, ref.render(*tens))


def test_frame_near_the_capacity_waits_for_its_count():
    print("[case] near the capacity", flush=True)
    ref, tens = _setup(1 << 20)
    want = ref.render(*tens)
    rast, _ = _setup(want.num_pairs)                 # fits exactly
    _same(rast.render(*tens), want)
    rast.lib.count.clear()
    grown = [t.clone() for t in tens]
    grown[1] *= 1.5                                  # larger surfels: more pairs than slots
    fr = rast.render(*grown)
    assert fr.num_pairs > want.num_pairs and rast.lib.count["fs_render_forward"] == 1
    _same(fr, ref.render(*grown))


@pytest.mark.parametrize("kw", [{}, {"topk": 4}])
def test_frame_that_jumps_past_its_buffers_is_taken_again(kw):
    print(f"[case] jump {kw}", flush=True)
    ref, tens = _setup(1 << 20, **kw)
    small = [t.clone() for t in tens]
    small[1] *= 0.1
    few, many = ref.render(*small).num_pairs, ref.render(*tens).num_pairs
    rast, _ = _setup((few * 8 + 6) // 7 + 8, **kw)
    assert rast.render(*small).num_pairs == few and few * 8 <= rast.capacity * 7 and many > rast.capacity
    rast.lib.count.clear()
    fr = rast.render(*tens)
    assert rast.lib.count["fs_render_forward"] == 2
    _same(fr, ref.render(*tens))
    _same(rast.render(*small), ref.render(*small))


def test_later_frames_make_no_events_or_buffers(monkeypatch):
    print("[case] no per-frame objects", flush=True)
    rast, tens = _setup(1 << 20)
    rast.render(*tens)
    made = []
    monkeypatch.setattr(torch.cuda, "Event", lambda *a, **k: made.append("event"))
    empty = torch.empty
    monkeypatch.setattr(torch, "empty", lambda *a, **k: (made.append("pinned") if k.get("pin_memory") else None,
                                                         empty(*a, **k))[1])
    for _ in range(3):
        rast.render(*tens)
    assert made == []
