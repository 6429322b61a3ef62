"""The one-launch re-sort of small sets whose keys did not change (a set at rest), or all but one
did not: the stable order of the new keys, the flags of the others, and no sort paid for."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import polypic_oracle as O
from tests.gpu_util import dev, host, note, oracle_grid, require_gpu
from tests.test_gpu_parity import _full_sort, _resort

pytestmark = pytest.mark.gpu


def sorted_set(pp, P, n):
    s = W.random_scene(P + n, n, P)
    g = pp.grid_from_spec(s.grid)
    keys, perm = _full_sort(pp, g, dev(s.x), P)
    return g, oracle_grid(g), s.x[:, host(perm)].copy(), keys


@pytest.mark.parametrize("n", [9, 300])  # 2 and 4 digits of key
@pytest.mark.parametrize("P", [1, 64, 65, 1025, 8192])
def test_unchanged_keys_keep_their_places(P, n):
    pp = require_gpu()
    note(f"small re-sort at rest: P={P} n={n}")
    g, og, x, keys = sorted_set(pp, P, n)
    keys2, perm2, status = _resort(pp, g, dev(x), keys, P)
    assert status == 0
    assert torch.equal(keys2, keys)
    assert np.array_equal(host(perm2), np.arange(P))


@pytest.mark.parametrize("P", [2, 64, 1025, 8192])
@pytest.mark.parametrize("at", ["first", "middle", "last"])
def test_one_changed_key_is_sorted_in(P, at):
    pp = require_gpu()
    note(f"small re-sort, {at} of {P} changed")
    g, og, x, keys = sorted_set(pp, P, 42)
    k = {"first": 0, "middle": P // 2, "last": P - 1}[at]
    x[:, k] = (2.5 + 38.0 * (x[:, k] < 0.5)) / 42  # the far corner
    keys2, perm2, status = _resort(pp, g, dev(x), keys, P)
    keys_ref, perm_ref = O.sort_keys(og, x)
    assert status == 0
    assert np.array_equal(host(keys2).view(np.uint32), keys_ref)
    assert np.array_equal(host(perm2), perm_ref)


@pytest.mark.parametrize("P", [2, 65, 8192])
def test_unchanged_keys_out_of_order_are_sorted_and_flagged(P):
    pp = require_gpu()
    note(f"small re-sort, {P} unchanged keys out of order")
    g, og, x, keys = sorted_set(pp, P, 42)
    x, keys = x[:, ::-1].copy(), keys.flip(0).contiguous()
    if int(keys[0]) == int(keys[-1]):
        pytest.skip("one cell")
    keys2, perm2, status = _resort(pp, g, dev(x), keys, P)
    keys_ref, perm_ref = O.sort_keys(og, x)
    assert status == pp._lib.POLYPIC_FLAG_ORDER
    assert np.array_equal(host(keys2).view(np.uint32), keys_ref)
    assert np.array_equal(host(perm2), perm_ref)


def test_a_set_at_rest_pays_for_no_pass():
    """8,192 slots, 4 digits: 10 us unchanged against 31 with every 30th changed (0.7 asked)."""
    pp = require_gpu()
    P, n = 8192, 300
    g, og, x, keys = sorted_set(pp, P, n)
    moved = x.copy()
    moved[0, ::30] = np.clip(moved[0, ::30] + np.float32(1.0 / n), 2.5 / n, (n + 1.5) / n)
    ws = torch.empty(pp.ops.polypic_sort_update_workspace_bytes(g, P), dtype=torch.uint8,
                     device="cuda")
    out, perm = torch.empty_like(keys), torch.empty_like(keys)

    def ms(pos):
        t = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                pp.ops.polypic_sort_update(g, pos, keys, out, perm, ws)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) / 20)
        return sorted(t)[5]

    rest, flow = dev(x), dev(moved)
    ms(rest)
    note(f"small re-sort: unchanged {ms(rest):.4f} ms, changed {ms(flow):.4f} ms")
    assert ms(rest) <= 0.7 * ms(flow)
