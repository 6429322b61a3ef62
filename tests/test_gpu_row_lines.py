"""Rows of a count that 16 does not divide, at 27 modes and past the size from which kernels
write them in whole lines: G2P, staggered and mixture G2P (with F), the fused call and the
P2G adjoint give the bits they give for the same particles in a set of an even count, whose
rows are written slot by slot.  (Its last particles are out of the way and not compared.)"""
import pytest
import torch

from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu

P_EVEN = 160 * 1024  # 16 divides it; 27 modes: 53 MB of rows


def fields(pp, P):
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    n = 32
    grid = pp.make_grid((n + 4,) * 3, 1.0 / n)
    N = (n + 4) ** 3
    rnd = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    x = ((3.0 + rnd(3, P_EVEN) * (n - 2)) / n)
    f = {"x": x, "gv": rnd(3 * N) - 0.5, "gv6": rnd(6 * N) - 0.5, "F": rnd(9, P_EVEN),
         "m": 0.5 + rnd(P_EVEN), "c": rnd(3, 27, P_EVEN) - 0.5, "gm": rnd(N) + 0.5,
         "gx": rnd(3, P_EVEN), "phase": (rnd(P_EVEN) < 0.4).int()}
    return grid, N, {k: (v[..., :P].contiguous() if v.shape[-1] == P_EVEN else v)
                     for k, v in f.items()}


def outputs(pp, op, P, bad):
    grid, N, f = fields(pp, P)
    if bad:
        f["x"][1, 1000:P_EVEN - 1000:997] = -3.0  # flagged and zeroed
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    full = lambda *s: torch.full(s, 7.0, device="cuda")  # noqa: E731
    co, xo, Fo, mo = full(3, 27, P), full(3, P), full(9, P), full(P)
    kw = dict(x_out=xo, F_in=f["F"], F_out=Fo, status_dev=status)
    if op == "g2p":
        pp.ops.polypic_g2p(grid, 27, 1e-3, f["gv"], f["x"], co, mass_in=f["m"], mass_out=mo, **kw)
    elif op == "mac":
        pp.ops.polypic_mac_g2p(grid, 27, 1e-3, f["gv"], f["x"], co, mass_in=f["m"], mass_out=mo,
                               **kw)
    elif op == "mixture":
        po = torch.zeros(P, dtype=torch.int32, device="cuda")
        pp.ops.polypic_mixture_g2p(grid, 27, 1e-3, f["gv6"], f["x"], f["phase"], co, phase_out=po,
                                   mass_f_in=f["m"], mass_f_out=mo, mass_s_in=f["m"],
                                   mass_s_out=torch.empty_like(mo), **kw)
        mo = mo + po
    elif op == "fused":
        gm, gp = torch.empty(N, device="cuda"), torch.empty(3 * N, device="cuda")
        pp.ops.polypic_g2p2g(grid, 27, 1e-3, f["gv"], f["x"], xo, co, gm, gp, F_in=f["F"],
                             F_out=Fo, mass_in=f["m"], mass_out=mo, status_dev=status)
    else:
        xo.zero_()
        pp.ops.polypic_p2g_backward(grid, 27, f["x"], f["c"], f["gm"], f["gv"], co, xo,
                                    mass=f["m"], mass_grad=mo, status_dev=status)
        Fo = xo
    torch.cuda.synchronize()
    assert bool(int(status.item()) & 1) == bad
    return co, xo, Fo, mo


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("cut", [1, 4, 24, 255, 256 + 97, 512 - 33])
@pytest.mark.parametrize("op", ["g2p", "mac", "mixture", "fused", "p2g_backward"])
def test_rows_in_whole_lines_equal_rows_by_slot(op, cut, bad):
    pp = require_gpu()
    P = P_EVEN - cut
    note(f"row lines: {op} P={P} out-of-range particles: {bad}")
    ref = outputs(pp, op, P_EVEN, bad)
    got = outputs(pp, op, P, bad)
    for a, b in zip(got, ref):
        assert torch.equal(a, b[..., :P])
