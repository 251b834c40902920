"""fs_sort orders the caller's pairs by (key, value), also where a list repeats a
pair (1,500 times: more than a part of the distribution takes): every copy keeps a place of its own.  Runs at the edges of the run sorts
(one wave, a workgroup's distribution, radix), bit-exact against a stable sort."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2604_10951_amd import _lib as L

pytestmark = pytest.mark.gpu

SIZES = (2, 64, 129, 256, 257, 300, 511, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193)


@pytest.mark.parametrize("depths", ["spread", "bunched"])
@pytest.mark.parametrize("copies", [2, 5, 60, 1500])
def test_repeated_pairs(depths, copies):
    print(f"[case] repeated pairs {depths} x{copies}", flush=True)
    rng = np.random.default_rng(copies)
    keys, vals = [], []
    for t, n in enumerate(SIZES):
        m = -(-n // copies)
        z = rng.uniform(1.0, 60.0, m) if depths == "spread" else 10.0 + 1e-3 * rng.standard_normal(m)
        if depths == "bunched":
            z[0] = 60.0
        k = (np.uint64(t) << np.uint64(32)) | z.astype(np.float32).view(np.uint32).astype(np.uint64)
        v = rng.integers(0, 1 << 20, m).astype(np.uint32)
        keys.append(np.tile(k, copies)[:n])
        vals.append(np.tile(v, copies)[:n])
    keys, vals = np.concatenate(keys), np.concatenate(vals)
    order = rng.permutation(len(keys))
    keys, vals = keys[order], vals[order]
    want = np.lexsort((vals, keys))
    lib, T, P = L.load(), len(SIZES), len(keys)
    k, v = torch.from_numpy(keys.view(np.int64)).cuda(), torch.from_numpy(vals.view(np.int32)).cuda()
    count = torch.tensor([P], dtype=torch.int64, device="cuda")
    ranges = torch.empty(2 * T, dtype=torch.int32, device="cuda")
    ws = torch.empty(lib.fs_workspace_bytes(0, 1, T, P, ctypes.byref(L.make_opts())), dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())   # noqa: E731
    L.check(lib.fs_sort(p(k), p(v), P, p(count), P, T, p(ranges), p(ws),
                        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)), "fs_sort")
    torch.cuda.synchronize()
    assert np.array_equal(k.cpu().numpy().view(np.uint64), keys[want])
    assert np.array_equal(v.cpu().numpy().view(np.uint32), vals[want])
