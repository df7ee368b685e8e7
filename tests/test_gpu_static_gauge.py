"""A static lapse or shift leaves the gauge source terms out: the right-hand
sides of the lapse and the shift do not see K and B^i at all, not even where
those are infinite or NaN, in every kernel that a stage can run in.
"""
import numpy as np
import pytest

from paper_1111_3344_amd import inputs as I

pytestmark = pytest.mark.gpu

N = (40, 12, 10)


@pytest.mark.parametrize("order", [4, 8])
@pytest.mark.parametrize("path,precision,thr,bc", [
    ("auto", 0, 0.3, I.BC_STATIC), ("auto", 0, 0.3, I.BC_PERIODIC),
    ("auto", 1, 0.0, I.BC_STATIC), ("auto", 1, np.inf, I.BC_STATIC),
    ("direct", 0, 0.3, I.BC_STATIC), ("direct", 1, 0.0, I.BC_STATIC),
    ("direct", 0, 0.3, I.BC_PERIODIC), ("direct", 1, 0.0, I.BC_PERIODIC)])
def test_sources_left_out(path, precision, thr, bc, order):
    import torch
    from paper_1111_3344_amd import bssn as B
    g = I.GridSpec(N, 5 if order == 8 else 3, (0.1, 0.11, 0.12),
                   (-0.7, -0.5, -0.6), bc)
    u = I.smooth_random(g, seed=5 + order)
    if bc == I.BC_PERIODIC:
        I.fill_periodic_ghosts(g, u)
    bad = u.copy()
    v = g.interior(bad)
    v[I.TRK, 3, 5, 7] = np.inf
    v[I.TRK, 8, 2, 33] = np.nan
    for i, s in enumerate((I.BX, I.BY, I.BZ)):
        v[s, 2 + i, 4, 20 + i] = (np.inf, -np.inf, np.nan)[i]
    print(f"[static gauge] {path} precision={precision} thr={thr} bc={bc} "
          f"order={order}", flush=True)
    prm = dict(fd_order=order, precision=precision, fp64_alpha_threshold=thr,
               eta_R=0.5)
    gauge = (I.ALP, I.BETX, I.BETY, I.BETZ)
    res = {}
    B.bssn_set_path(B.BSSN_PATH_DIRECT if path == "direct"
                    else B.BSSN_PATH_AUTO)
    try:
        for fixed in (0, 1):
            for name, x in (("good", u), ("bad", bad)):
                du = torch.from_numpy(x).to("cuda")
                out = torch.zeros_like(du)
                B.bssn_rhs(g, B.Params(lapse_static=fixed, shift_static=fixed,
                                       **prm), du, out)
                res[fixed, name] = g.interior(out.cpu().numpy())
    finally:
        B.bssn_set_path(B.BSSN_PATH_AUTO)
    for s in gauge:
        assert np.isfinite(res[1, "good"][s]).all()
        assert np.array_equal(res[1, "good"][s], res[1, "bad"][s]), s
        # a live gauge does see them
        assert not np.isfinite(res[0, "bad"][s]).all(), s
