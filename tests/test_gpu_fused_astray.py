"""The fused G2P2G where a chunk's particles move apart: a few of a tile fast while the others
rest, or the others fast while a few rest, by more cells than a brick's margin.  The chunk's
bricks are then placed by the slots they hold; what no brick holds goes to HBM.

Each half against the oracle, as the other tests of the call; every node the scatter filled lies
in a flagged region.
"""
import numpy as np
import pytest
import torch

from oracle import polypic_oracle as O
from tests.gpu_util import TOL_NORMWISE, dev, host, note, oracle_grid, rel, require_gpu, ulp_ok
from tests.test_gpu_active import filled_nodes, region_ids, unpack
from tests.test_gpu_fused_bricks import scene

pytestmark = pytest.mark.gpu

KINDS = ["jet", "rest", "splash", "shear", "everywhere"]


def velocity(kind, cells, shape, n, rng):
    """Node velocities (3, N, N, N) that move particles by up to `cells` cells in dt = 1."""
    v = np.zeros((3,) + shape, np.float32)
    if kind == "jet":       # through the middle of the first cell of every tile
        v[0, 1::4, 1::4, 1::4] = cells
    elif kind == "rest":    # everything but those cells
        v[0] = cells
        v[0, 1::4, 1::4, 1::4] = -1.37 * cells
    elif kind == "splash":  # a few nodes, any direction
        at = rng.random(shape) < 0.03
        v[:, at] = rng.uniform(-cells, cells, (3, int(at.sum())))
    elif kind == "shear":   # from one layer of nodes to the next
        v[0] = cells * ((np.arange(shape[1]) % 3) - 1)[None, :, None]
    else:                   # every node its own way: no brick holds many
        v[:] = rng.uniform(-cells, cells, v.shape)
    return v / np.float32(n)


@pytest.mark.parametrize("n_modes", [1, 4, 8, 27])
@pytest.mark.parametrize("cells", [1.5, 3.0, 9.0])
@pytest.mark.parametrize("kind", KINDS)
def test_particles_that_move_apart(kind, cells, n_modes):
    pp = require_gpu()
    case = {"jet": "at_rest", "rest": "dense_16", "splash": "mixed", "shear": "sparse",
            "everywhere": "at_rest"}[kind]
    spec, x, c, mass, F, _ = scene(case, None, 11, True)
    P = x.shape[1]
    note(f"fused astray: {kind} {cells} n_modes={n_modes} P={P}")
    g = pp.grid_from_spec(spec)
    og = oracle_grid(g)
    ps = pp.ParticleSet(g, n_modes, dev(x), dev(c[:, :n_modes]), dt=1.0, bc_layers=0,
                        gravity=(0.0, 0.0, 0.0), mass=dev(mass), F=dev(F))
    ps.sort()
    gv = velocity(kind, cells, (og.nz, og.ny, og.nx), spec.cells[0], np.random.default_rng(7))
    ps.grid_vel.copy_(dev(gv).reshape(-1))
    ps.region_state.zero_()
    src = host(ps.perm)
    ps.g2p2g()
    torch.cuda.synchronize()
    assert ps.status_flags() == 0
    c_ref, x_ref, F_ref = O.g2p(og, gv.astype(np.float64), x[:, src], n_modes, 1.0, F[:, src])
    c_new = host(ps.coeff_next).reshape(3, n_modes, P)
    assert rel(c_new, c_ref) <= TOL_NORMWISE
    assert ulp_ok(host(ps.x_next), x_ref, 2, 1.5)
    assert rel(host(ps.F_next), F_ref) <= 1e-6
    M_ref, Q_ref = O.p2g(og, host(ps.x_next), c_new, n_modes, mass[src])
    assert rel(host(ps.grid_mass).reshape(M_ref.shape), M_ref) <= TOL_NORMWISE
    assert rel(host(ps.grid_mom).reshape(Q_ref.shape), Q_ref) <= TOL_NORMWISE
    flags = unpack(ps.region_state, pp.ops.polypic_region_count(g))
    N = g.nx * g.ny * g.nz
    need = np.unique(region_ids(g.nx, g.ny, g.nz, filled_nodes(ps.grid_mass, ps.grid_mom, N)))
    assert (flags[need] != 0).all()


def test_a_jet_leaves_the_others_in_their_bricks():
    """A set at rest but for the first cell of every tile, which moves 3 cells: the call takes 1.1
    times as long as at rest where those alone leave their bricks, and 2.8 times where a brick
    goes with its first particle and the others are added to HBM (2.5 times asked; 1.3 and 7 at
    4.19 M particles)."""
    pp = require_gpu()
    n, m = 64, 4
    cells = torch.cartesian_prod(*[torch.arange(48, device="cuda")] * 3).t().repeat_interleave(
        8, 1)
    P = cells.shape[1]
    rng = torch.Generator("cuda").manual_seed(3)
    x = (10.0 + cells + torch.rand(3, P, device="cuda", generator=rng)) / n
    ps = pp.ParticleSet(pp.make_grid((n + 4,) * 3, 1.0 / n), m, x,
                        torch.zeros(3, m, P, device="cuda"), dt=1.0)
    ps.sort()

    def ms(jump):
        v = torch.zeros(3, n + 4, n + 4, n + 4, device="cuda")
        v[0, 1::4, 1::4, 1::4] = jump * 2.37 / n  # (the weight at a cell's middle is 0.42)
        ps.grid_vel.copy_(v.reshape(-1))
        t = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ps.g2p2g()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return sorted(t)[4]

    ms(0.0)
    note(f"fused jet: rest {ms(0.0):.4f} ms, 3 cells {ms(3.0):.4f} ms")
    assert ms(3.0) <= 2.5 * ms(0.0)


@pytest.mark.parametrize("n_modes", [1, 4, 8, 27])
@pytest.mark.parametrize("tiles", [(256,), (255, 1), (100, 156), (3, 200, 53), (64, 64, 64, 64),
                                   (1, 1, 1, 253), (40,) * 6 + (16,), (256, 100, 156, 37)])
def test_chunks_of_one_tile_and_more(tiles, n_modes):
    """Chunks whose slots lie in one tile (one round of the scatter, all channels), in two or
    three (two rounds), and in more than there are bricks; at the grid's corner and inside it."""
    pp = require_gpu()
    note(f"fused rounds: {tiles} n_modes={n_modes}")
    n = 40
    rng = np.random.default_rng(sum(tiles) + n_modes)
    corner = [(4 * (k % 3), 4 * (k // 3), 4 * (k % 2)) for k in range(len(tiles))]
    x = np.concatenate([(1.0 + np.array(corner[k])[:, None] + 3.98 * rng.random((3, m)))
                        for k, m in enumerate(tiles)], 1)
    x = (np.maximum(x, 2.001) / n).astype(np.float32)
    P, N = x.shape[1], n + 4
    g = pp.make_grid((N,) * 3, 1.0 / n)
    og = oracle_grid(g)
    gv = (0.05 * rng.uniform(-1, 1, (3, N, N, N)) / n).astype(np.float32)
    f = lambda *s: torch.full(s, 7.0, device="cuda")  # noqa: E731
    xo, co, gm, gp = f(3, P), f(3, n_modes, P), f(N ** 3), f(3 * N ** 3)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    pp.ops.polypic_g2p2g(g, n_modes, 1.0, dev(gv).reshape(-1), dev(x), xo, co, gm, gp,
                         status_dev=st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    c_ref, x_ref, _ = O.g2p(og, gv.astype(np.float64), x, n_modes, 1.0)
    assert rel(host(co), c_ref) <= TOL_NORMWISE
    M_ref, Q_ref = O.p2g(og, host(xo), host(co), n_modes)
    assert rel(host(gm).reshape(M_ref.shape), M_ref) <= TOL_NORMWISE
    assert rel(host(gp).reshape(Q_ref.shape), Q_ref) <= TOL_NORMWISE


@pytest.mark.parametrize("n_modes", [4, 27])
@pytest.mark.parametrize("chunks", [256, 257])
@pytest.mark.parametrize("past", [64, 65])
def test_slots_without_a_brick_in_small_launches(past, chunks, n_modes):
    """Chunks of four tiles whose last one, past the bricks, holds a quarter of the slots or one
    more: the bricks are placed anew for either in a launch of 257 workgroups, and only for more
    than a quarter in one of 256."""
    pp = require_gpu()
    note(f"fused small launch: {past} past the bricks, {chunks} chunks, n_modes={n_modes}")
    n = 40
    rng = np.random.default_rng(past + chunks + n_modes)
    t = np.repeat(np.arange(4 * chunks) % 512, np.tile([64, 64, 128 - past, past], chunks))
    tile = 4.0 * np.stack([t % 8, t // 8 % 8, t // 64])
    x = np.maximum(1.0 + tile + 3.98 * rng.random((3, len(t))), 2.001)
    x = (x / n).astype(np.float32)
    P, N = x.shape[1], n + 4
    g = pp.make_grid((N,) * 3, 1.0 / n)
    og = oracle_grid(g)
    gv = (0.05 * rng.uniform(-1, 1, (3, N, N, N)) / n).astype(np.float32)
    f = lambda *s: torch.full(s, 7.0, device="cuda")  # noqa: E731
    xo, co, gm, gp = f(3, P), f(3, n_modes, P), f(N ** 3), f(3 * N ** 3)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    pp.ops.polypic_g2p2g(g, n_modes, 1.0, dev(gv).reshape(-1), dev(x), xo, co, gm, gp,
                         status_dev=st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    c_ref, x_ref, _ = O.g2p(og, gv.astype(np.float64), x, n_modes, 1.0)
    assert rel(host(co), c_ref) <= TOL_NORMWISE
    assert ulp_ok(host(xo), x_ref, 2, 1.5)
    M_ref, Q_ref = O.p2g(og, host(xo), host(co), n_modes)
    assert rel(host(gm).reshape(M_ref.shape), M_ref) <= TOL_NORMWISE
    assert rel(host(gp).reshape(Q_ref.shape), Q_ref) <= TOL_NORMWISE
