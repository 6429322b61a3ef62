"""The fused G2P2G's base node of positions whose u lies within a rounding of a cell's border.

u = (x - o) inv_dx rounds up to the border where the product alone is below it, so a floor of
the rounded product and a floor that fuses the product into the subtraction differ.  Every
kernel of the library takes the fused one: the fused call has to give the state that the G2P
call gives (the coefficients jump with the stencil from cell to cell) and to refuse and accept
the positions that it refuses and accepts.
"""
import numpy as np
import pytest
import torch

from tests.gpu_util import note, rel, require_gpu, host

CELLS = 100


def borders(nodes):
    """Positions (as float32) at the cell borders of the axis where the two floors differ, and
    the base node of the fused one."""
    inv = np.float32(CELLS)
    at = (np.arange(nodes) + 0.5) / CELLS
    near = [at.astype(np.float32)]
    for to in (-9, 9):
        near.append(np.nextafter(near[0], np.float32(to)))
    x = np.unique(np.concatenate(near))
    rounded = np.floor((x * inv).astype(np.float32) - np.float32(0.5))
    # (the product of two float32 and the subtraction are exact in 64 bits)
    fused = np.floor((x.astype(np.float64) * inv - 0.5).astype(np.float32))
    pick = rounded != fused
    return x[pick], fused[pick]


def test_there_are_such_borders():
    x, base = borders(CELLS + 4)
    assert {4.0, 16.0, 32.0} <= set(base + 1)
    assert -1.0 in base  # accepted by the one, refused by the other


def calls(pp, x, n_modes, nodes):
    g = pp.make_grid((nodes,) * 3, 1.0 / CELLS)
    P, N = x.shape[1], nodes ** 3
    x = torch.from_numpy(x).cuda()
    gv = torch.randn(3 * N, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    f = lambda *s: torch.full(s, 7.0, device="cuda")  # noqa: E731
    out = []
    for call in ("g2p", "fused"):
        st = torch.zeros(1, dtype=torch.int32, device="cuda")
        c, xo = f(3, n_modes, P), f(3, P)
        if call == "g2p":
            pp.ops.polypic_g2p(g, n_modes, 1e-4, gv, x, c, x_out=xo, status_dev=st)
        else:
            pp.ops.polypic_g2p2g(g, n_modes, 1e-4, gv, x, xo, c, f(N), f(3 * N), status_dev=st)
        torch.cuda.synchronize()
        out.append((host(c), host(xo), int(st.item())))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("n_modes", [1, 4, 8, 27])
def test_fused_state_equals_g2p_at_cell_borders(n_modes):
    pp = require_gpu()
    nodes = CELLS + 4
    x1, base = borders(nodes)
    x1 = x1[base >= 1]
    note(f"fused offsets: n_modes={n_modes} borders at {x1 * CELLS}")
    rng = np.random.default_rng(2)
    P = 700
    x = ((3.0 + 90.0 * rng.random((3, P))) / CELLS).astype(np.float32)
    for a in range(3):
        at = rng.integers(0, 3, P) == 0
        x[a, at] = rng.choice(x1, int(at.sum()))
    (c0, x0, st0), (c, xn, st) = calls(pp, x, n_modes, nodes)
    assert st0 == 0 and st == 0
    assert rel(c, c0) <= 1e-6  # (the same sums; a stencil one cell off changes it by O(1))
    assert np.array_equal(xn, x0) or np.max(np.abs(xn - x0)) <= 2 * np.spacing(np.float32(1))


@pytest.mark.gpu
@pytest.mark.parametrize("edge", ["low", "high"])
def test_fused_call_refuses_and_accepts_what_g2p_does(edge):
    """At the low edge the fused floor gives base node -1 (refused); at the high edge of a grid
    of 34 nodes base node 31, the last (accepted), where the rounded product gives 32."""
    pp = require_gpu()
    x1, base = borders(CELLS + 4)
    nodes = CELLS + 4 if edge == "low" else 34
    xe = x1[base == (-1.0 if edge == "low" else 31.0)][:1]
    assert xe.size == 1
    x = np.full((3, 300), 10.2 / CELLS, np.float32)
    x[1, ::7] = xe
    note(f"fused offsets: {edge} edge at {xe * CELLS}")
    (c0, _, st0), (c, _, st) = calls(pp, x, 27, nodes)
    assert st0 == (1 if edge == "low" else 0)
    assert st == st0
    assert rel(c, c0) <= 1e-6
