"""Mixed precision with every tile in FP64 (an infinite threshold) is the FP64
method bitwise, also where a whole tile's lapse is NaN, infinite or above 1e300:
each tile is written by one of the two launches, single and batched.
"""
import numpy as np
import pytest

from paper_1111_3344_amd import inputs as I

pytestmark = pytest.mark.gpu

# whole tiles, tiles cut by the grid's end, one tile
SIZES = [(40, 14, 11), (64, 48, 40), (16, 4, 4)]


def _state(n, order, value):
    """A smooth state whose lapse is `value` over the last tile (with the
    remainders of n) and over one tile in the middle."""
    g = I.GridSpec(n, 5 if order == 8 else 3, (0.1, 0.11, 0.12),
                   (-0.7, -0.5, -0.6), I.BC_STATIC)
    u = I.smooth_random(g, seed=sum(n) + order)
    a = g.interior(u)[I.ALP]
    for o in ([(m - 1) // t * t for m, t in zip(n, (16, 4, 4))],
              [m // 2 // t * t for m, t in zip(n, (16, 4, 4))]):
        a[o[2]:o[2] + 4, o[1]:o[1] + 4, o[0]:o[0] + 16] = value
    return g, u


def _both(order):
    from paper_1111_3344_amd import bssn as B
    return (B.Params(fd_order=order),
            B.Params(fd_order=order, precision=B.BSSN_MIXED,
                     fp64_alpha_threshold=np.inf))


@pytest.mark.parametrize("order", [4, 8])
@pytest.mark.parametrize("value", [np.nan, np.inf, 2e300])
@pytest.mark.parametrize("n", SIZES)
def test_rhs_is_fp64(n, value, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    g, u = _state(n, order, value)
    print(f"[threshold] n={n} lapse={value} order={order}", flush=True)
    du = torch.from_numpy(u).to("cuda")
    out = []
    for prm in _both(order):
        o = torch.full_like(du, 7.0)
        B.bssn_rhs(g, prm, du, o)
        out.append(g.interior(o.cpu().numpy()))
    assert not (out[1] == 7.0).any()
    assert np.array_equal(out[0], out[1], equal_nan=True)


@pytest.mark.parametrize("order", [4, 8])
@pytest.mark.parametrize("value", [np.nan, 2e300])
def test_batched_step_is_fp64(value, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    sets = [_state(n, order, value) for n in SIZES]
    grids = [g for g, _ in sets]
    print(f"[threshold] batched lapse={value} order={order}", flush=True)
    res = []
    for prm in _both(order):
        u = [torch.from_numpy(x).to("cuda") for _, x in sets]
        bufs = [u] + [[t.clone() for t in u] for _ in range(3)]
        plan = B.batch_patches_plan(grids, prm, *bufs, 0.01, autotune=0)
        assert all(c[1:] == (16, 4, 4) for c in B.batch_patches_describe(plan))
        B.batch_patches(plan, 1)
        res.append([g.interior(t.cpu().numpy()) for g, t in zip(grids, u)])
        plan.destroy()
    for a, b, (g, x) in zip(*res, sets):
        assert np.array_equal(a, b, equal_nan=True)
        # the step was taken: no value of the smooth slots is left as it was
        assert not (b[I.PHI] == g.interior(x)[I.PHI]).any()
