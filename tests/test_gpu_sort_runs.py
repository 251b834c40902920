"""fs_sort on runs at the edges of its run sorts (one wave up to 256 entries, a
workgroup's distribution over the depth range up to 2,048 and 8,192, radix
beyond) with depths that spread, bunch or repeat: bunched ones do not fit the
distribution and take the network.  Bit-exact against a stable sort."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2604_10951_amd import _lib as L

pytestmark = pytest.mark.gpu

SIZES = (0, 1, 64, 65, 128, 129, 255, 256, 257, 511, 1023, 1024, 1025, 2047, 2048, 2049, 4100, 8191, 8192, 8193)


def _depths(rng, n, kind):
    if kind == "spread":
        z = rng.normal(23.0, 1.0, n).astype(np.float32)
    elif kind == "equal":
        z = np.full(n, 7.25, np.float32)
    elif kind == "bunched":    # most entries within a few ulps, some far away
        z = np.float32(22.0) + (rng.integers(0, 6, n) * np.float32(2e-6)).astype(np.float32)
        z[rng.random(n) < 0.02] = 1e4
    else:                      # a mixture of repeated planes and noise
        z = np.where(rng.random(n) < 0.5, np.float32(3.0) + rng.integers(0, 40, n).astype(np.float32),
                     rng.uniform(0.3, 90.0, n).astype(np.float32)).astype(np.float32)
    return z.view(np.uint32).astype(np.uint64)


@pytest.mark.parametrize("kind", ["spread", "equal", "bunched", "planes"])
def test_sort_runs(kind):
    print(f"[case] sort runs {kind}", flush=True)
    rng = np.random.default_rng(5)
    tiles = rng.permutation(len(SIZES) * 3)[:len(SIZES)]     # some tiles stay empty
    keys = np.concatenate([(np.uint64(t) << np.uint64(32)) | _depths(rng, n, kind) for t, n in zip(tiles, SIZES)])
    vals = rng.permutation(len(keys)).astype(np.uint32)
    order = rng.permutation(len(keys))
    keys, vals = keys[order], vals[order]
    want = np.lexsort((vals, keys))
    lib, T, P = L.load(), len(SIZES) * 3, len(keys)
    cap = P + 100
    k = torch.zeros(cap, dtype=torch.int64, device="cuda")
    v = torch.zeros(cap, dtype=torch.int32, device="cuda")
    k[:P] = torch.from_numpy(keys.view(np.int64)).cuda()
    v[:P] = torch.from_numpy(vals.view(np.int32)).cuda()
    count = torch.tensor([P], dtype=torch.int64, device="cuda")
    ranges = torch.empty(2 * T, dtype=torch.int32, device="cuda")
    ws = torch.empty(lib.fs_workspace_bytes(0, 1, T, cap, ctypes.byref(L.make_opts())), dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())   # noqa: E731
    st = lib.fs_sort(p(k), p(v), cap, p(count), -1, T, p(ranges), p(ws),
                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    L.check(st, "fs_sort")
    torch.cuda.synchronize()
    assert np.array_equal(k[:P].cpu().numpy().view(np.uint64), keys[want])
    assert np.array_equal(v[:P].cpu().numpy().view(np.uint32), vals[want])
    r = ranges.cpu().numpy().reshape(T, 2)
    n = np.bincount((keys >> np.uint64(32)).astype(np.int64), minlength=T)
    assert np.array_equal(r[:, 1] - r[:, 0], n) and np.array_equal(r[:, 0], np.cumsum(n) - n)
