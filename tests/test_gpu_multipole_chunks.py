"""Multipoles where the launches split: one node, fewer points than a wave,
around 64 points per interpolation workgroup and 1,024 per chunk, the largest
|spin| and l, against the oracle.

Tolerance: 1e-11 of the largest coefficient for l <= 8, 1e-8 at l = 16, where
Goldberg's sum cancels about 4^l / l of its largest term.
"""
import numpy as np
import pytest

from oracle import multipole as MP
from paper_1111_3344_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,nph,spin,lmax", [
    (1, 1, 0, 2), (2, 3, -1, 3), (3, 21, 2, 4), (5, 13, -2, 4),
    (8, 128, -2, 4), (25, 41, 8, 8), (25, 41, -8, 8), (33, 97, -2, 8),
    (64, 70, 3, 16)])
def test_matches_oracle(nt, nph, spin, lmax):
    from paper_1111_3344_amd import bssn as B
    g = I.GridSpec((18, 14, 16), 3, (0.11, 0.12, 0.1), (-0.9, -0.8, -0.75))
    u = I.smooth_random(g, seed=nt)
    re, im = (g.view(u)[s] for s in (0, 7))
    c, r = (0.02, -0.03, 0.01), 0.5
    want = np.asarray(MP.multipole(g, re, im, c, r, spin, lmax, nt, nph))
    print(f"[multipole] {nt} x {nph} spin {spin} lmax {lmax}", flush=True)
    du = B.to_device(u)
    got = B.bssn_multipole(g, du, du, c, r, spin, lmax, nt, nph, im_slot=7)
    tol = 1e-11 if lmax <= 8 else 1e-8
    assert np.abs(got - want).max() <= tol * np.abs(want).max()
