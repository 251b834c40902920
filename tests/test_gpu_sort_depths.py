"""fs_sort of long runs however their depths are spread: the distribution cuts equal
parts of the depth range, or the intervals between samples where those crowd.
Run lengths at the edges of its forms, many runs of the shortest (sorted four at a
time), bit-exact against a stable sort."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2604_10951_amd import _lib as L

pytestmark = pytest.mark.gpu

KINDS = {
    "normal": lambda rng, n: rng.normal(23.0, 1.0, n),
    "wall": lambda rng, n: np.where(rng.random(n) < 0.02, rng.uniform(11, 60, n), 10 + 1e-3 * rng.standard_normal(n)),
    "planes": lambda rng, n: rng.integers(1, 12, n) * 1.5,
    "two": lambda rng, n: np.where(rng.random(n) < 0.5, 3.0, 50.0),
    "equal": lambda rng, n: np.full(n, 7.25),
    "outlier": lambda rng, n: np.where(np.arange(n) == n // 2, 1e30, 10 + 1e-4 * rng.standard_normal(n)),
    "wide": lambda rng, n: np.exp(rng.uniform(-80, 80, n)),
}
RUNS = [257] * 700 + [511, 512] * 500 + [513, 600, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4097, 8191, 8192, 8193]


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("kind", list(KINDS))
def test_depths(kind, many):
    print(f"[case] sort depths {kind} many={many}", flush=True)
    rng = np.random.default_rng(len(kind) + many)
    runs = RUNS if many else RUNS[-15:]
    z = np.concatenate([KINDS[kind](rng, n) for n in runs]).astype(np.float32)
    keys = (np.repeat(np.arange(len(runs), dtype=np.uint64), runs) << np.uint64(32)) | z.view(np.uint32)
    order = rng.permutation(len(keys))
    keys, vals = keys[order], rng.permutation(len(keys)).astype(np.uint32)
    want = np.lexsort((vals, keys))
    lib, T, P = L.load(), len(runs), len(keys)
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
