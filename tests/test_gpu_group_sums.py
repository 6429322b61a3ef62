"""What a lane group of the fused G2P2G and of the mixture P2G adds up before the 64-bit bricks,
in chunks of dense cells (10 particles per cell and more), where four lanes may stand for one
atomic: two neighbours are added in 32 bits, the two sums in 64 bits, and a value that is not
finite reaches no further than its lane's partner."""
import numpy as np
import pytest
import torch

from oracle import polypic_oracle as O
from tests.gpu_util import dev, host, note, oracle_grid, rel, require_gpu

pytestmark = pytest.mark.gpu

N = 32
CALLS = ["fused", "fused_quads", "batch", "mixture"]


def scatter(pp, call, n_modes, x, mass, c):
    """Grid mass and momentum that the call scatters from particles at rest (the mixture: with
    the coefficients c), in the caller's order."""
    g = pp.make_grid((N + 4,) * 3, 1.0 / N)
    nodes, P = (N + 4) ** 3, x.shape[1]
    f = lambda *s: torch.zeros(s, device="cuda")  # noqa: E731
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    gm, gp = f(nodes), f(3 * nodes)
    if call == "mixture":
        gm, gp = f(2 * nodes), f(6 * nodes)
        pp.ops.polypic_mixture_p2g(g, n_modes, dev(x), torch.zeros(P, dtype=torch.int32,
                                                                   device="cuda"), dev(mass),
                                   dev(c), gm, gp, status_dev=st)
        gm, gp = gm[:nodes], gp[:3 * nodes]
    else:
        # a velocity of 1 at every node: mode 0 is 1 and the others vanish (to rounding)
        kw = dict(mass_in=dev(mass), status_dev=st)
        gv, xo, co = f(3 * nodes) + 1.0, f(3, P), f(3, n_modes, P)
        if call == "batch":
            pp.ops.polypic_batch_g2p2g(pp.ops.Batch([(g, P)]), n_modes, 0.0, gv, dev(x), xo, co,
                                       gm, gp, **kw)
        else:
            pp.ops.polypic_set_g2p2g_config(n_modes, 4 if call == "fused_quads" else -1, -1)
            try:
                pp.ops.polypic_g2p2g(g, n_modes, 0.0, gv, dev(x), xo, co, gm, gp, **kw)
            finally:
                pp.ops.polypic_set_g2p2g_config(n_modes, -1, -1)
        c = host(co)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    shape = (N + 4,) * 3
    return oracle_grid(g), host(gm).reshape(shape), host(gp).reshape((3,) + shape), c


@pytest.mark.parametrize("n_modes", [1, 4, 8, 27])
@pytest.mark.parametrize("call", CALLS)
def test_large_values_that_cancel_leave_the_small_ones(call, n_modes):
    """32 particles at one place, (M, M, 1, 1, -M, -M, 1, 1) and so on: the pairs' sums are exact
    doubles of a value and the large ones cancel in the brick.  What is left is 16 small values,
    each rounded once or a few times in 32 bits (relative error 2e-7 per stage of the weights;
    1e-6 asked): a 32-bit sum of a large and a small pair would lose M 2^-24, 6 % of them."""
    pp = require_gpu()
    note(f"group sums: {call} n_modes={n_modes}")
    x = np.repeat(np.array([[10.3], [9.75], [11.2]], np.float32) / np.float32(N), 32, axis=1)
    mass = np.tile(np.array([1, 1, 2**-20, 2**-20, -1, -1, 2**-20, 2**-20], np.float32) * 2**20, 4)
    rng = np.random.default_rng(1)
    c = np.repeat(rng.standard_normal((3, n_modes, 1)).astype(np.float32), 32, axis=2)
    og, gm, gp, c = scatter(pp, call, n_modes, x, mass, c)
    small = np.abs(mass) == 1.0
    M, Q = O.p2g(og, x[:, small], c[:, :, small], n_modes, mass[small])
    assert rel(gm, M) <= 1e-6
    assert rel(gp, Q) <= 1e-6


@pytest.mark.parametrize("n_modes", [4, 27])
@pytest.mark.parametrize("call", ["fused", "batch", "mixture"])
def test_a_nan_stays_with_its_cell(call, n_modes):
    """10 particles in one cell, then 12 in another, far from it; one of the first cell's last
    pair has a NaN mass.  Its four lanes hold a pair of either cell: the second cell's nodes get
    what its particles give."""
    pp = require_gpu()
    note(f"group sums: NaN, {call} n_modes={n_modes}")
    x = np.empty((3, 22), np.float32)
    x[:, :10] = 8.3 / N
    x[:, 10:] = 14.6 / N
    mass = np.ones(22, np.float32)
    mass[8] = np.nan
    c = np.full((3, n_modes, 22), 0.5, np.float32)
    og, gm, gp, c = scatter(pp, call, n_modes, x, mass, c)
    assert np.isnan(gm).any()
    M, Q = O.p2g(og, x[:, 10:], c[:, :, 10:], n_modes, mass[10:])
    at = M != 0
    assert rel(gm[at], M[at]) <= 1e-6
    assert rel(gp[:, at], Q[:, at]) <= 1e-6


@pytest.mark.parametrize("n_modes", [1, 4, 8, 27])
@pytest.mark.parametrize("base", [(1, 0, 0), (0, 0, 0), (5, 2, 1)])
def test_a_pair_beside_two_single_lanes(base, n_modes):
    """Four slots of the mixture P2G (in the caller's order) that hold two particles of one cell
    and one each of two other cells, in a chunk of dense cells, in its second tile: the pair is
    added by itself.  (Base node (1, 0, 0) in the second brick is where a lane that reads its own
    register in place of an idle neighbour's finds its own cell and brick.)"""
    pp = require_gpu()
    note(f"group sums: pair and singles at {base}, n_modes={n_modes}")
    at = lambda b: (np.array(b, np.float32) + np.float32(1.0)) / N  # noqa: E731
    far, one, two = (20, 20, 20), (9, 9, 9), (17, 9, 9)
    cells = [far] * 128 + [base, base, one, two] + [one] * 124
    x = np.ascontiguousarray(np.stack([at(b) for b in cells], 1).astype(np.float32))
    rng = np.random.default_rng(4)
    c = rng.standard_normal((3, n_modes, 256)).astype(np.float32)
    mass = (0.5 + rng.random(256)).astype(np.float32)
    og, gm, gp, _ = scatter(pp, "mixture", n_modes, x, mass, c)
    M, Q = O.p2g(og, x, c, n_modes, mass)
    assert rel(gm, M) <= 1e-5
    here = tuple(slice(v, v + 3) for v in base[::-1])
    assert rel(gm[here], M[here]) <= 1e-6
    assert rel(gp[(slice(None),) + here], Q[(slice(None),) + here]) <= 1e-5


@pytest.mark.parametrize("put_back", [False, True])
def test_a_setting_read_and_put_back_keeps_the_default(put_back):
    """The default takes quads in chunks of dense cells, and so does the setting that get reports
    for it: 16 per cell, 1 mode, where pairs throughout take 1.3 times as long (1.2 asked)."""
    pp = require_gpu()
    ops = pp.ops
    note(f"group setting read and put back: {put_back}")
    n, ppc, m = 64, 16, 1
    rng = torch.Generator("cuda").manual_seed(3)
    cells = torch.cartesian_prod(*[torch.arange(40, device="cuda")] * 3).t().repeat_interleave(
        ppc, 1)
    P = cells.shape[1]
    x = (12.0 + cells + torch.rand(3, P, device="cuda", generator=rng)) / n
    ps = pp.ParticleSet(pp.make_grid((n + 4,) * 3, 1.0 / n), m, x,
                        torch.zeros(3, m, P, device="cuda"), dt=0.0)
    ps.sort()

    def ms(lane_group):
        ops.polypic_set_g2p2g_config(m, lane_group, -1)
        t = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ps.g2p2g()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return sorted(t)[4]

    try:
        ms(-1)
        got = ops.polypic_get_g2p2g_config(m)
        again = got.lane_group if put_back else -1
        assert ms(again) <= 1.2 * ms(-1)
        assert ms(again) <= 1.2 * ms(4)
    finally:
        ops.polypic_set_g2p2g_config(m, -1, -1)
