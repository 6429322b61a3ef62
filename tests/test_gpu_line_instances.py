"""The kernels that write 27-mode rows in whole lines, each instance of them, whole outputs: the
fused call (rows' ends through the caches, and streamed from 4.0 M particles on) with a sort
permutation, its grid sums too, and the batched G2P with scenes that begin inside a workgroup.

Sizes are just past the size from which the rows are written so (48 MB of them) and either side
of the change to streamed ends.  The fused call is compared with the G2P call and with the P2G
call on its outputs (each against the oracle in tests of its own): coefficients and sums of 32-bit
products in another order, 1e-6 normwise."""
import numpy as np
import pytest
import torch

from oracle import polypic_oracle as O
from tests.gpu_util import TOL_NORMWISE, host, note, oracle_grid, rel, require_gpu

pytestmark = pytest.mark.gpu


def relative(a, b):
    """Normwise, on the device in 64 bits."""
    a, b = a.double(), b.double()
    return float((a - b).norm() / b.norm())


def block(P, n, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    side = int(np.ceil((P / 8) ** (1 / 3)))
    at = torch.arange(P, device="cuda") // 8
    cell = torch.stack([at % side, (at // side) % side, at // side ** 2])
    x = (3.0 + cell + torch.rand(3, P, device="cuda", generator=g)) / n
    assert side + 4 <= n
    return x.contiguous(), g


# 155,353, 155,356 and 155,360 + 8: rows start off the 32 bytes, at 16 of them, and at 32 (by slot)
@pytest.mark.parametrize("P", [155_353, 155_356, 155_368, 3_999_999, 4_000_001, 4_000_004,
                               (1 << 22) + 5])
def test_fused_rows_and_sums(P):
    pp = require_gpu()
    ops, n = pp.ops, 32 if P < 1 << 20 else 96
    note(f"line instances: fused P={P}")
    grid = pp.make_grid((n + 4,) * 3, 1.0 / n)
    N = (n + 4) ** 3
    x, g = block(P, n, P)
    rnd = lambda *s: torch.rand(*s, device="cuda", generator=g)  # noqa: E731
    gv = (rnd(3 * N) - 0.5) / n
    mass, F = 0.5 + rnd(P), rnd(9, P)
    keys, perm = (torch.empty(P, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.empty(ops.polypic_sort_workspace_bytes(grid, P), dtype=torch.uint8, device="cuda")
    ops.polypic_sort(grid, x, keys, perm, ws)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    new = lambda *s: torch.full(s, 7.0, device="cuda")  # noqa: E731
    co, xo, Fo, mo, gm, gp = new(3, 27, P), new(3, P), new(9, P), new(P), new(N), new(3 * N)
    ops.polypic_g2p2g(grid, 27, 0.5, gv, x, xo, co, gm, gp, perm=perm, F_in=F, F_out=Fo,
                      mass_in=mass, mass_out=mo, status_dev=st)
    c1, x1, F1 = new(3, 27, P), new(3, P), new(9, P)
    ops.polypic_g2p(grid, 27, 0.5, gv, x, c1, perm=perm, x_out=x1, F_in=F, F_out=F1,
                    status_dev=st)
    assert relative(co, c1) <= 1e-6
    assert float((xo - x1).abs().max()) <= 2 * np.spacing(np.float32(1.0))
    assert relative(Fo, F1) <= 1e-6
    assert torch.equal(mo, mass[perm.long()])
    del c1, x1, F1
    m1, p1 = new(N), new(3 * N)
    ops.polypic_p2g(grid, 27, xo, co, m1, p1, mass=mo, status_dev=st)
    assert int(st.item()) == 0
    assert relative(gm, m1) <= 1e-6
    assert relative(gp, p1) <= 1e-6
    if P < 1 << 20:  # and the oracle's sums
        og = oracle_grid(grid)
        M, Q = O.p2g(og, host(xo), host(co), 27, host(mo))
        assert rel(host(gm).reshape(M.shape), M) <= TOL_NORMWISE
        assert rel(host(gp).reshape(Q.shape), Q) <= TOL_NORMWISE


@pytest.mark.parametrize("counts", [(100_003, 55_352), (1, 511, 513, 160_000, 0, 37, 2),
                                    (40_001,) * 4, (155_360 + 8,)])
@pytest.mark.parametrize("with_perm", [False, True])
def test_batched_g2p_rows(counts, with_perm):
    """Every scene's rows, to the bit, as the G2P call gives them for the scene alone."""
    pp = require_gpu()
    ops = pp.ops
    note(f"line instances: batch {counts} perm {with_perm}")
    sizes = (32, 28, 34, 40, 24, 26, 30)
    xs, gvs, scenes, single = [], [], [], []
    for k, P in enumerate(counts):
        n = sizes[k]
        grid = pp.make_grid((n + 4,) * 3, 1.0 / n)
        x, g = block(P, n + 8, k) if P else (torch.empty(3, 0, device="cuda"), None)
        gv = torch.rand(3 * (n + 4) ** 3, device="cuda",
                        generator=torch.Generator("cuda").manual_seed(k)) - 0.5
        x = x * (n + 8) / n if P else x
        x = x.clamp(2.5 / n, (n + 1.0) / n).contiguous()
        perm = torch.randperm(P, device="cuda", generator=g).int() if P else None
        c, xo = torch.empty(3, 27, P, device="cuda"), torch.empty(3, P, device="cuda")
        if P:
            ops.polypic_g2p(grid, 27, 1e-3, gv, x, c, perm=perm if with_perm else None, x_out=xo)
        xs.append(x)
        gvs.append(gv)
        scenes.append((grid, P))
        single.append((c, xo, perm))
    b = ops.Batch(scenes)
    off = np.cumsum((0,) + counts)
    perm = torch.cat([s[2] + int(o) for s, o in zip(single, off) if s[2] is not None]).int()
    # grid arrays: component major over all scenes' nodes
    gv = torch.cat([v.reshape(3, -1) for v in gvs], 1).reshape(-1).contiguous()
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    co = torch.full((3, 27, b.P), 7.0, device="cuda")
    xo = torch.full((3, b.P), 7.0, device="cuda")
    ops.polypic_batch_g2p(b, 27, 1e-3, gv, torch.cat(xs, 1).contiguous(), co,
                          perm=perm if with_perm else None, x_out=xo, status_dev=st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    for k, P in enumerate(counts):
        sl = slice(int(off[k]), int(off[k + 1]))
        assert torch.equal(co[:, :, sl], single[k][0])
        assert torch.equal(xo[:, sl], single[k][1])
