"""Frames whose per-block launches would pass 2^32 threads are refused before anything
is enqueued (host checks only: no pointer is read)."""
from __future__ import annotations

import ctypes

import pytest

from paper_2604_10951_amd import _lib as L

HIP_ERROR_INVALID_VALUE = 1


@pytest.mark.parametrize("topk_mode", [L.FS_TOPK_FIRST, L.FS_TOPK_WEIGHT])
@pytest.mark.parametrize("tile,tiles", [(8, 1 << 24), (32, 1 << 20)])
def test_split_render_of_too_many_blocks_is_refused(tile, tiles, topk_mode):
    lib = L.load()
    o = L.make_opts(tile=tile, topk=1, schedule=L.FS_SCHED_SPLIT, topk_mode=topk_mode)
    p = ctypes.c_void_p(4096)   # never dereferenced
    st = lib.fs_render_forward(p, None, p, p, p, 4, 100, p, 1, tiles, ctypes.byref(o), p, p, p, None, None, None, None,
                               None, p, None)
    assert st == L.FS_ERR_HIP and lib.fs_last_hip_error() == HIP_ERROR_INVALID_VALUE
    st = lib.fs_render_labels(p, p, p, p, 4, 100, p, 1, tiles, ctypes.byref(o), p, None, p, p, None, p, None)
    assert st == L.FS_ERR_HIP and lib.fs_last_hip_error() == HIP_ERROR_INVALID_VALUE
