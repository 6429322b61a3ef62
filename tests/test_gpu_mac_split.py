"""The staggered P2G on either side of the size up to which a workgroup takes one component (131,072
particles): its face sums are those of its halves (each well below that size, against the oracle in
tests of their own)."""
import pytest
import torch

from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


def particles(P, n, n_modes, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    rnd = lambda *s: torch.rand(*s, device="cuda", generator=g)  # noqa: E731
    return (3.0 + (n - 4) * rnd(3, P)) / n, rnd(3, n_modes, P) - 0.5, 0.5 + rnd(P)


@pytest.mark.parametrize("n_modes", [1, 4, 8, 27])
@pytest.mark.parametrize("P", [131_071, 131_072, 131_073, 131_329])
def test_sums_are_those_of_the_halves(P, n_modes):
    pp = require_gpu()
    note(f"mac split: P={P} n_modes={n_modes}")
    n = 24
    N = (n + 4) ** 3
    grid = pp.make_grid((n + 4,) * 3, 1.0 / n)
    x, c, m = particles(P, n, n_modes, P)
    keys, perm = (torch.empty(P, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.empty(pp.ops.polypic_sort_workspace_bytes(grid, P), dtype=torch.uint8, device="cuda")
    pp.ops.polypic_sort(grid, x, keys, perm, ws)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    whole = torch.zeros(3 * N, device="cuda"), torch.zeros(3 * N, device="cuda")
    halves = torch.zeros(3 * N, device="cuda"), torch.zeros(3 * N, device="cuda")
    pp.ops.polypic_mac_p2g(grid, n_modes, x, c, *whole, mass=m, perm=perm, status_dev=st)
    for at in (perm[:P // 2].long(), perm[P // 2:].long()):
        pp.ops.polypic_mac_p2g(grid, n_modes, x[:, at].contiguous(), c[:, :, at].contiguous(),
                               *halves, mass=m[at], accumulate=True, status_dev=st)
    assert int(st.item()) == 0
    for a, b in zip(whole, halves):
        for k in range(3):  # every component by itself
            a1, b1 = a[k * N:(k + 1) * N].double(), b[k * N:(k + 1) * N].double()
            assert float((a1 - b1).norm() / b1.norm()) <= 1e-6
