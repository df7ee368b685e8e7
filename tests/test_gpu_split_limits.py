"""The split stage kernels at the ends of their loops.

  * The FP64 pass of mixed precision looks at 64 tiles of a workgroup at a time
    per wave and at 512 per round: grids with more than either (one point wide, so
    that a tile has 16 points), single and batched.  A tile with one low lapse
    is bitwise the FP64 right-hand side, the others are not.
  * The smallest periodic grids that are accepted (the stencil's reach, with an
    even number of points in x), where a box wraps several times, against the
    oracle to 1e-12 of each slot's largest value, as for the larger ones.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1111_3344_amd import inputs as I

pytestmark = pytest.mark.gpu


class Narrow(I.GridSpec):
    """Rows padded to an even length only."""

    @property
    def sy(self):
        return -(-self.ext[0] // 2) * 2


def _narrow(ny, nz, order):
    ghost = 5 if order == 8 else 3
    return Narrow((1, ny, nz), ghost, (0.1, 0.11, 0.12), (0.3, -0.5, -0.6),
                  I.BC_STATIC)


def _interior(g, t):
    v = t[g.off0:g.off0 + 25 * g.sf].view(25, g.ext[2], g.ext[1], g.sy)
    k = g.ghost
    return v[:, k:k + g.n[2], k:k + g.n[1], k:k + g.n[0]]


def _state(g, seed):
    """Noise around flat space with a lapse of 0.9, and 0.49 at one point of
    every tenth tile or so; whether each (z, y) tile has one."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.rand(g.total, generator=gen, device="cuda",
                   dtype=torch.float64).mul_(0.01)
    v = u[g.off0:].view(25, g.sf)
    for s in (I.GXX, I.GYY, I.GZZ):
        v[s] += 1.0
    v[I.ALP] += 0.9
    nt = [(g.n[a] + 3) // 4 for a in (2, 1)]
    low = torch.rand(nt, generator=gen, device="cuda") < 0.1
    low[-1, -1] = True
    z, y = (i.cpu().numpy() for i in torch.nonzero(low, as_tuple=True))
    rng = np.random.default_rng(seed)
    z = np.minimum(4 * z + rng.integers(0, 4, len(z)), g.n[2] - 1)
    y = np.minimum(4 * y + rng.integers(0, 4, len(y)), g.n[1] - 1)
    _interior(g, u)[I.ALP][torch.from_numpy(z), torch.from_numpy(y), 0] = 0.49
    return u, low


def _tiles_equal(g, a, b):
    import torch
    import torch.nn.functional as F
    eq = (_interior(g, a) == _interior(g, b)).all(0).all(-1)
    eq = F.pad(eq.to(torch.uint8), (0, -g.n[1] % 4, 0, -g.n[2] % 4), value=1)
    return eq.view(-(-g.n[2] // 4), 4, -(-g.n[1] // 4), 4).amin((1, 3)) == 1


# 67 tiles per workgroup of 256; 521 of them
@pytest.mark.parametrize("ny,nz,order", [(522, 519, 4), (522, 519, 8),
                                         (1480, 1441, 4)])
def test_scan_of_many_tiles(ny, nz, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    g = _narrow(ny, nz, order)
    u, low = _state(g, ny + order)
    print(f"[scan] {ny} x {nz} order={order}", flush=True)
    out = []
    for prm in (B.Params(fd_order=order),
                B.Params(fd_order=order, precision=B.BSSN_MIXED,
                         fp64_alpha_threshold=0.5)):
        o = torch.zeros_like(u)
        B.bssn_rhs(g, prm, u, o)
        out.append(o)
    assert torch.equal(_tiles_equal(g, *out), low)


@pytest.mark.parametrize("ny,nz,order", [(522, 519, 4), (522, 519, 8),
                                         (1480, 1441, 4)])
def test_batched_scan_of_many_tiles(ny, nz, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    grids = [_narrow(9, 6, order), _narrow(ny, nz, order),
             _narrow(50, 61, order)]
    us = [_state(g, 7 + i)[0] for i, g in enumerate(grids)]
    prm = B.Params(fd_order=order, precision=B.BSSN_MIXED,
                   fp64_alpha_threshold=0.5)
    dt = 1e-4
    print(f"[scan] batched {ny} x {nz} order={order}", flush=True)
    bufs = [[u.clone() for u in us] for _ in range(4)]
    plan = B.batch_patches_plan(grids, prm, *bufs, dt, autotune=0)
    B.batch_patches(plan, 1)
    torch.cuda.synchronize()
    plan.destroy()
    for g, u, got in zip(grids, us, bufs[0]):
        a, b, acc = u.clone(), u.clone(), torch.zeros_like(u)
        one = u.clone()
        B.rk4_step(g, prm, dt, one, a, b, acc)
        assert torch.isfinite(_interior(g, one)).all()
        assert torch.equal(one, got)


@pytest.mark.parametrize("n,order", [((4, 3, 3), 4), ((4, 5, 3), 4),
                                     ((6, 3, 4), 4), ((20, 3, 3), 4),
                                     ((6, 5, 5), 8), ((8, 6, 5), 8),
                                     ((22, 5, 7), 8), ((18, 9, 5), 8)])
def test_smallest_periodic(n, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    g = I.GridSpec(n, 5 if order == 8 else 3, (0.1, 0.11, 0.12),
                   (-0.7, -0.5, -0.6), I.BC_PERIODIC)
    u = I.smooth_random(g, seed=sum(n) + order)
    I.fill_periodic_ghosts(g, u)
    print(f"[periodic] n={n} order={order}", flush=True)
    v = np.full_like(u, np.nan)        # the device copy has no ghosts
    g.interior(v)[...] = g.interior(u)
    du = torch.from_numpy(v).to("cuda")
    out = torch.zeros_like(du)
    B.bssn_rhs(g, B.Params(fd_order=order), du, out)
    k = g.interior(O.rhs(g, O.params(fd_order=order), u)).reshape(25, -1)
    got = g.interior(out.cpu().numpy()).reshape(25, -1)
    d = np.abs(k).max(1)
    d = np.where(d > 0, d, d.max())
    assert (np.abs(got - k).max(1) / d).max() <= 1e-12
