"""The one-launch sort of small sets on the GPU (up to 8,192 particles), at the sizes around its
rounds and its limit: the full sort and the re-sort give the oracle's stable argsort, for one
scene and for a batch, and raise the flags that the larger sort raises."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import polypic_oracle as O
from tests.gpu_util import dev, host, note, oracle_grid, require_gpu
from tests.test_gpu_parity import _full_sort, _resort

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 1023, 1024, 1025, 2049, 7169, 8191, 8192, 8193]


@pytest.mark.parametrize("n", [9, 42, 300])  # 2, 3 and 4 digits of key
@pytest.mark.parametrize("P", SIZES)
def test_small_sorts_match_the_oracle(P, n):
    pp = require_gpu()
    s = W.random_scene(P, n, P)
    g = pp.grid_from_spec(s.grid)
    og = oracle_grid(g)
    note(f"small sort: P={P} n={n}")
    keys, perm = _full_sort(pp, g, dev(s.x), P)
    keys_ref, perm_ref = O.sort_keys(og, s.x)
    assert np.array_equal(host(keys).view(np.uint32), keys_ref)
    assert np.array_equal(host(perm), perm_ref)
    rng = np.random.default_rng(P)
    xs = s.x[:, perm_ref].copy()
    pick = rng.random(P) < 0.3
    xs[0, pick] += np.float32(1.0 / n)
    keys2, perm2, status = _resort(pp, g, dev(xs), keys, P)
    keys_ref, perm_ref = O.sort_keys(og, xs)
    assert status == 0
    assert np.array_equal(host(keys2).view(np.uint32), keys_ref)
    assert np.array_equal(host(perm2), perm_ref)


@pytest.mark.parametrize("P", [3, 1000, 8192])
def test_small_sort_flags(P):
    pp = require_gpu()
    s = W.random_scene(3, 20, P)
    g = pp.grid_from_spec(s.grid)
    note(f"small sort flags: P={P}")
    keys, perm = _full_sort(pp, g, dev(s.x), P)
    xs = s.x[:, host(perm)].copy()
    shuffled = keys.flip(0).contiguous()
    keys2, perm2, status = _resort(pp, g, dev(xs), shuffled, P)
    assert status == pp._lib.POLYPIC_FLAG_ORDER
    xs[1, P // 2] = -3.0
    keys2, perm2, status = _resort(pp, g, dev(xs), keys, P)
    assert status == pp._lib.POLYPIC_FLAG_RANGE
    assert np.array_equal(np.sort(host(perm2)), np.arange(P))
    assert (np.diff(host(keys2).view(np.uint32).astype(np.int64)) >= 0).all()


@pytest.mark.parametrize("counts", [(1, 0, 5), (700, 64, 1300, 2), (3000, 0, 5192), (4000, 4193)])
def test_small_batch_sorts_match_each_scene(counts):
    pp = require_gpu()
    sizes = (16, 40, 23, 64)
    scenes = [W.random_scene(k, sizes[k], c) for k, c in enumerate(counts)]
    grids = [pp.grid_from_spec(s.grid) for s in scenes]
    b = pp.ops.Batch([(g, c) for g, c in zip(grids, counts)])
    P = sum(counts)
    note(f"small batch sort: {counts}")
    x = np.concatenate([s.x for s in scenes], axis=1)
    keys = torch.empty(P, dtype=torch.int32, device="cuda")
    perm = torch.empty_like(keys)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(1, pp.ops.polypic_batch_sort_workspace_bytes(b)), dtype=torch.uint8,
                     device="cuda")
    pp.ops.polypic_batch_sort(b, dev(x), keys, perm, ws, status)
    ref = np.concatenate([o + O.sort_keys(oracle_grid(g), s.x)[1] if c else np.empty(0, int)
                          for g, s, c, o in zip(grids, scenes, counts,
                                                np.cumsum((0,) + counts[:-1]))])
    assert np.array_equal(host(perm), ref)
    xs = x[:, ref]
    keys2, perm2 = torch.empty_like(keys), torch.empty_like(perm)
    ws2 = torch.empty(pp.ops.polypic_batch_sort_update_workspace_bytes(b), dtype=torch.uint8,
                      device="cuda")
    pp.ops.polypic_batch_sort_update(b, dev(xs), keys, keys2, perm2, ws2, status)
    assert np.array_equal(host(perm2), np.arange(P))
    assert torch.equal(keys, keys2)
    assert int(status.item()) == 0
