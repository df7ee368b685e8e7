"""The split stage kernels (curvature and transport waves) at the sizes where
they can go wrong: partial tiles in every direction, one tile, one tile per
workgroup, several tiles per workgroup (the pipeline across tiles), each stage
of the update, FP64 and mixed precision, against the oracle's right-hand side.

Tolerances: an FP64 right-hand side agrees with the oracle to 1e-12 of each
slot's largest value (rounding of about 5,000 operations per point, as in the
parity tests); mixed precision to 1e-5.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1111_3344_amd import inputs as I

pytestmark = pytest.mark.gpu

# one point; one tile; a remainder in each direction; 480 tiles on 256
# workgroups (one and two tiles each); 2,080 tiles (eight and nine)
SIZES = [(1, 1, 1), (16, 4, 4), (17, 5, 6), (63, 9, 3), (64, 48, 40),
         (80, 61, 101)]


def _grid(n, ghost):
    return I.GridSpec(n, ghost, (0.1, 0.11, 0.12), (-0.7, -0.5, -0.6),
                      I.BC_STATIC)


def _err(g, got, ref):
    a, b = (g.interior(x).reshape(25, -1) for x in (got, ref))
    d = np.abs(b).max(1)
    return (np.abs(a - b).max(1) / np.where(d > 0, d, max(d.max(), 1e-300)))


@pytest.mark.parametrize("order", [4, 8])
@pytest.mark.parametrize("n", SIZES)
def test_rhs_and_stages(n, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    g = _grid(n, 5 if order == 8 else 3)
    u = I.smooth_random(g, seed=sum(n) + order)
    print(f"[split] n={n} order={order}", flush=True)
    k = O.rhs(g, O.params(fd_order=order), u)
    du = torch.from_numpy(u).to("cuda")
    out = torch.zeros_like(du)
    prm = B.Params(fd_order=order)
    B.bssn_rhs(g, prm, du, out)
    assert _err(g, out.cpu().numpy(), k).max() <= 1e-12
    mixed = torch.zeros_like(du)
    B.bssn_rhs(g, B.Params(fd_order=order, precision=B.BSSN_MIXED), du, mixed)
    assert _err(g, mixed.cpu().numpy(), k).max() <= 1e-5
    # each stage's update from the same stage input
    un = I.smooth_random(g, seed=91)
    acc0 = I.smooth_random(g, seed=92)
    dt = 0.01
    for s, (wa, wo) in enumerate(((dt / 6, dt / 2), (dt / 3, dt / 2),
                                  (dt / 3, dt), (0.0, dt / 6))):
        acc = torch.from_numpy(acc0).to("cuda")
        o = torch.zeros_like(du)
        B.rk4_stage(g, prm, s, dt, torch.from_numpy(un).to("cuda"), du, acc,
                    o)
        base = acc0 if s == 3 else un
        # increments, so that the stored sums' own rounding counts against
        # the value (1e-15) and the right-hand side against the increment
        for got, b, w in ((o, base, wo),
                          (acc, un if s == 0 else acc0, wa)):
            d = g.interior(got.cpu().numpy()) - g.interior(b)
            ref = w * g.interior(k)
            tol = (1e-12 * np.abs(ref).reshape(25, -1).max(1) +
                   4e-16 * np.abs(g.interior(b)).reshape(25, -1).max(1) +
                   4e-16 * np.abs(ref).reshape(25, -1).max(1))
            assert (np.abs(d - ref).reshape(25, -1).max(1) <= tol).all(), s


# periodic grids on the same kernel: x extents below, at and above a tile
# (even: whole granules wrap; odd: the direct kernel), y and z below the
# tile and the stencil's reach, several tiles per workgroup
@pytest.mark.parametrize("order", [4, 8])
@pytest.mark.parametrize("n", [(6, 5, 5), (16, 4, 6), (18, 7, 9), (17, 8, 8),
                               (32, 32, 32), (48, 50, 46)])
def test_periodic_rhs_and_step(n, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    n = tuple(max(v, 5) for v in n) if order == 8 else n
    g = I.GridSpec(n, 5 if order == 8 else 3, (0.1, 0.11, 0.12),
                   (-0.7, -0.5, -0.6), I.BC_PERIODIC)
    u = I.smooth_random(g, seed=sum(n) + order)
    I.fill_periodic_ghosts(g, u)
    print(f"[split] periodic n={n} order={order}", flush=True)
    # the device copy's ghosts are never read
    v = u.copy()
    g.view(v)[...] = np.nan
    g.interior(v)[...] = g.interior(u)
    du = torch.from_numpy(v).to("cuda")
    out = torch.zeros_like(du)
    prm = B.Params(fd_order=order)
    B.bssn_rhs(g, prm, du, out)
    k = O.rhs(g, O.params(fd_order=order), u)
    assert _err(g, out.cpu().numpy(), k).max() <= 1e-12
    a, b, acc = du.clone(), du.clone(), torch.zeros_like(du)
    ref = O.rk4_step(g, O.params(fd_order=order), 0.02, u)
    B.rk4_step(g, prm, 0.02, du, a, b, acc)
    inc = g.interior(du.cpu().numpy()) - g.interior(u)
    want = g.interior(ref) - g.interior(u)
    D = np.abs(want).reshape(25, -1).max(1)
    D = np.where(D > 0, D, D.max())
    # four right-hand sides, each to 1e-12 of its own scale
    assert (np.abs(inc - want).reshape(25, -1).max(1) / D).max() <= 1e-11
