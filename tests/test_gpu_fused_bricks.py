"""The fused G2P2G on the GPU where its bricks, lane groups and row writes change course:
particles that leave their tile (into the brick's outer cells, or past them: HBM), chunks
with more tiles than bricks, dense cells (quads by themselves), and rows that start off the
memory sectors (27 modes; counts from a few slots to several chunks, with mass and F).

Each half against the oracle, as the other tests of the call: G2P of the same grid velocity,
and P2G of the state the device wrote; every node the scatter filled lies in a flagged region.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import polypic_oracle as O
from tests.gpu_util import TOL_NORMWISE, dev, host, note, oracle_grid, rel, require_gpu, ulp_ok
from tests.test_gpu_active import filled_nodes, region_ids, unpack

pytestmark = pytest.mark.gpu

# (cells per axis of the grid, block of cells, particles per cell, largest displacement in cells)
CASES = {
    "at_rest": (24, (12, 9, 10), 8, 0.0),
    "cross_cells": (24, (12, 9, 10), 8, 0.9),        # into the outer cells of a brick
    "cross_bricks": (24, (12, 9, 10), 8, 4.5),       # past them: HBM
    "sparse": (40, (36, 36, 36), 1, 0.9),            # more tiles in a chunk than bricks
    "dense_16": (16, (6, 5, 7), 16, 0.9),            # quads
    "dense_40": (16, (3, 4, 3), 40, 0.5),
    "mixed": (24, (10, 10, 10), 11, 0.9),            # around the change to quads
    "translate": (32, (10, 9, 10), 8, 0.6),          # and all by DRIFT: the bricks move along
    "translate_dense": (32, (6, 5, 7), 16, 0.6),
}
DRIFT = (3.2, -4.7, 2.1)  # cells


def scene(case, P, seed, mass_f):
    n, dims, ppc, move = CASES[case]
    rng = np.random.default_rng(seed)
    g = W.cubic_grid(n)
    total = dims[0] * dims[1] * dims[2] * ppc
    P = total if P is None else min(P, total)
    lo = np.array([(n - d) // 2 for d in dims])[:, None]
    cells = np.stack(np.unravel_index(np.arange(total) // ppc, dims))
    x = ((2.0 + lo + cells + rng.random((3, total))) / n).astype(np.float32)[:, :P]
    c = rng.standard_normal((3, 27, P)).astype(np.float32)
    c[:, 1:] *= 0.1
    mass = (0.5 + rng.random(P)).astype(np.float32) if mass_f else None
    F = None
    if mass_f:
        F = (0.01 * rng.standard_normal((9, P))).astype(np.float32)
        F[::4] += 1.0
    return g, x, c, mass, F, move / n


def check(case, P, n_modes, mass_f, seed):
    pp = require_gpu()
    spec, x, c, mass, F, move = scene(case, P, seed, mass_f)
    P = x.shape[1]
    note(f"fused bricks: {case} P={P} n_modes={n_modes} mass and F: {mass_f}")
    g = pp.grid_from_spec(spec)
    og = oracle_grid(g)
    ps = pp.ParticleSet(g, n_modes, dev(x), dev(c[:, :n_modes]), dt=1.0, bc_layers=0,
                        gravity=(0.0, 0.0, 0.0), mass=None if mass is None else dev(mass),
                        F=None if F is None else dev(F))
    ps.sort()
    ps.p2g()
    ps.grid_update()
    # node velocities that move a particle by at most `move` per axis in dt = 1
    ps.grid_vel.uniform_(-move, move)
    if case.startswith("translate"):
        drift = torch.tensor(DRIFT, device="cuda")[:, None] / CASES[case][0]
        ps.grid_vel.copy_((ps.grid_vel.reshape(3, -1) + drift).reshape(-1))
    ps.region_state.zero_()
    torch.cuda.synchronize()
    gv = host(ps.grid_vel).reshape(3, og.nz, og.ny, og.nx).astype(np.float64)
    src = host(ps.perm)
    ps.g2p2g()
    torch.cuda.synchronize()
    assert ps.status_flags() == 0
    c_ref, x_ref, F_ref = O.g2p(og, gv, x[:, src], n_modes, 1.0, None if F is None else F[:, src])
    c_new = host(ps.coeff_next).reshape(3, n_modes, P)
    if move:
        assert rel(c_new, c_ref) <= TOL_NORMWISE
    else:
        assert not c_new.any()
    assert ulp_ok(host(ps.x_next), x_ref, 2, 1.5)
    if F is not None:
        assert rel(host(ps.F_next), F_ref) <= 1e-6
        assert np.array_equal(host(ps.mass_next), mass[src])
    M_ref, Q_ref = O.p2g(og, host(ps.x_next), c_new, n_modes,
                         None if mass is None else mass[src])
    assert rel(host(ps.grid_mass).reshape(M_ref.shape), M_ref) <= TOL_NORMWISE
    if move:
        assert rel(host(ps.grid_mom).reshape(Q_ref.shape), Q_ref) <= TOL_NORMWISE
    flags = unpack(ps.region_state, pp.ops.polypic_region_count(g))
    N = g.nx * g.ny * g.nz
    need = np.unique(region_ids(g.nx, g.ny, g.nz, filled_nodes(ps.grid_mass, ps.grid_mom, N)))
    assert (flags[need] != 0).all()


@pytest.mark.parametrize("n_modes", [1, 4, 8, 27])
@pytest.mark.parametrize("case", sorted(CASES))
def test_moving_particles_and_cell_densities(case, n_modes):
    check(case, None, n_modes, False, 11)


# one slot to several chunks; 8632 = 8 * 1079 and 8608 = 32 * 269 start rows on sectors
@pytest.mark.parametrize("P", [1, 2, 31, 32, 33, 63, 64, 95, 225, 255, 257, 287, 511, 2049, 8608,
                               8632, 8637])
def test_rows_off_the_sectors(P):
    check("cross_cells", P, 27, P % 2 == 1, P)


@pytest.mark.parametrize("n_modes", [8, 27])
def test_the_new_state_does_not_depend_on_the_lane_groups(n_modes):
    """Dense cells on a spacing that is no power of two, where a contracted product would
    round the offsets differently: pairs, quads and the default write the same bits."""
    pp = require_gpu()
    spec, x, c, mass, F, move = scene("dense_16", None, 5, True)
    spec = W.cubic_grid(42)
    x = (x * np.float32(16 / 42)).astype(np.float32)
    g = pp.grid_from_spec(spec)
    out = []
    for group in (2, 4, -1):
        pp.ops.polypic_set_g2p2g_config(n_modes, group, -1)
        try:
            ps = pp.ParticleSet(g, n_modes, dev(x), dev(c[:, :n_modes]), mass=dev(mass), F=dev(F),
                                dt=1e-3)
            ps.sort()
            ps.grid_vel.copy_(torch.linspace(-1, 1, ps.grid_vel.numel(), device="cuda"))
            ps.g2p2g()
            torch.cuda.synchronize()
        finally:
            pp.ops.polypic_set_g2p2g_config(n_modes, -1, -1)
        assert ps.status_flags() == 0
        out.append([host(t).copy() for t in (ps.x_next, ps.coeff_next, ps.F_next, ps.mass_next)])
    for other in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(out[0], other))


@pytest.mark.parametrize("n_modes", [4, 27])
@pytest.mark.parametrize("case", ["cross_cells", "dense_16", "dense_40", "mixed"])
def test_mixture_scatter_at_pairs_and_quads(case, n_modes):
    """The mixture P2G over cells on either side of the change to quads, both phases in the
    same cells: each phase against the oracle's P2G of its particles."""
    pp = require_gpu()
    spec, x, c, _, _, _ = scene(case, None, 3, False)
    P = x.shape[1]
    note(f"mixture groups: {case} P={P} n_modes={n_modes}")
    rng = np.random.default_rng(8)
    phase = (rng.random(P) < 0.3).astype(np.int32)
    mf, ms = rng.random((2, P)).astype(np.float32) + 0.5
    g = pp.grid_from_spec(spec)
    og = oracle_grid(g)
    ps = pp.MixtureParticleSet(g, n_modes, dev(x), dev(c[:, :n_modes]), dev(phase, torch.int32),
                               dev(mf), dev(ms), dt=1e-3)
    ps.sort()
    ps.p2g()
    torch.cuda.synchronize()
    assert ps.status_flags() == 0
    N = g.nx * g.ny * g.nz
    for k in range(2):
        at = phase == k
        m = (mf + ms if k else mf)[at]
        M_ref, Q_ref = O.p2g(og, x[:, at], c[:, :n_modes][:, :, at], n_modes, m)
        assert rel(host(ps.grid_mass).reshape(2, N)[k].reshape(M_ref.shape), M_ref) <= TOL_NORMWISE
        assert rel(host(ps.grid_mom).reshape(2, 3 * N)[k].reshape(Q_ref.shape), Q_ref) <= TOL_NORMWISE
