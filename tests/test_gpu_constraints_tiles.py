"""The constraint monitor's LDS kernel at the sizes where it can go wrong: one
point, one tile, remainders in each direction, grids thin in z (which take the
direct kernel), wider ghosts, orders 4 and 8, against the oracle.

Tolerance: 1e-12 of each field's largest value and of the norms (rounding of
about 2,000 operations on O(1) fields).
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1111_3344_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,ghost", [(4, 3), (4, 5), (8, 5)])
@pytest.mark.parametrize("n", [(1, 1, 1), (16, 4, 4), (17, 5, 6), (33, 7, 4),
                               (70, 9, 1), (64, 33, 12), (40, 38, 29)])
def test_fields_and_norms(n, order, ghost):
    import torch
    from paper_1111_3344_amd import bssn as B
    g = I.GridSpec(n, ghost, (0.1, 0.11, 0.12), (-0.7, -0.5, -0.6),
                   I.BC_STATIC)
    u = I.smooth_random(g, seed=sum(n))
    print(f"[constraints] n={n} order={order} ghost={ghost}", flush=True)
    centres = ((0.1, 0.0, 0.1),)
    H, M, G, want = O.constraints(g, O.params(fd_order=order), u, centres,
                                  0.25)
    du = torch.from_numpy(u).to("cuda")
    out = [torch.zeros_like(du) for _ in range(3)]
    norms = torch.zeros(8, dtype=torch.float64, device="cuda")
    B.bssn_constraints(g, B.Params(fd_order=order), du, norms, *out,
                       centres=centres, r_exc=0.25)
    for t, ref, k in zip(out, (H, M, G), (1, 3, 3)):
        a, b = (g.interior(x)[:k] for x in (t.cpu().numpy(), ref))
        assert np.abs(a - b).max() <= 1e-12 * max(np.abs(b).max(), 1e-300)
        # nothing outside the interior, nor beyond the field's slots
        t = t.cpu().numpy().copy()
        g.interior(t)[:k] = 0.0
        assert not t.any()
    got = norms.cpu().numpy()
    assert got[6] == want[6] and got[7] == want[7] == 0
    assert np.all(np.abs(got - want) <= 1e-12 * np.abs(want))
