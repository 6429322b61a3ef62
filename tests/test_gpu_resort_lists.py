"""Re-sorts whose list of changed pairs is around the length where their placement changes from a
pair per wavefront to a pair per lane: the exact stable order of the new keys."""
import numpy as np
import pytest
import torch

from oracle import polypic_oracle as O
from tests.gpu_util import dev, host, note, oracle_grid, require_gpu
from tests.test_gpu_parity import _full_sort, _resort

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("changed", [1, 63, 4032, 4095, 4096, 4097, 4159, 4161, 8192, 8193])
def test_resort_with_a_list_of(changed):
    pp = require_gpu()
    n, P = 60, 150_001
    note(f"re-sort of {P} with {changed} changed")
    rng = np.random.default_rng(changed)
    x = ((2.0 + 50.0 * rng.random((3, P))) / n).astype(np.float32)
    g = pp.make_grid((n + 4,) * 3, 1.0 / n)
    keys, perm = _full_sort(pp, g, dev(x), P)
    x = x[:, host(perm)].copy()
    at = rng.choice(P, changed, replace=False)
    x[1, at] += np.float32(3.0 / n)  # another cell for each of them
    keys2, perm2, status = _resort(pp, g, dev(x), keys, P)
    keys_ref, perm_ref = O.sort_keys(oracle_grid(g), x)
    assert status == 0
    assert np.array_equal(host(keys2).view(np.uint32), keys_ref)
    assert np.array_equal(host(perm2), perm_ref)
