"""Large spheres, whose Gauss-Legendre nodes are a launch of their own: on both
sides of the rule (33,024 points x 256 nodes is just above it, 32,895 x 255 just
below) and with the most nodes, against the oracle; and the cost of a point does
not grow with the number of nodes.

Tolerance: 1e-11 of the largest coefficient, as for the other spheres with
l <= 8.
"""
import ctypes

import numpy as np
import pytest

from oracle import multipole as MP
from paper_1111_3344_amd import inputs as I

pytestmark = pytest.mark.gpu

G = I.GridSpec((18, 14, 16), 3, (0.11, 0.12, 0.1), (-0.9, -0.8, -0.75))


@pytest.mark.parametrize("nt,nph", [(255, 129), (256, 129), (1024, 40)])
def test_matches_oracle(nt, nph):
    from paper_1111_3344_amd import bssn as B
    u = I.smooth_random(G, seed=nt)
    re, im = (G.view(u)[s] for s in (0, 7))
    c, r = (0.02, -0.03, 0.01), 0.5
    want = np.asarray(MP.multipole(G, re, im, c, r, -2, 3, nt, nph))
    print(f"[multipole] {nt} x {nph}", flush=True)
    du = B.to_device(u)
    got = B.bssn_multipole(G, du, du, c, r, -2, 3, nt, nph, im_slot=7)
    assert np.abs(got - want).max() <= 1e-11 * np.abs(want).max()


def test_cost_per_point():
    import torch
    from paper_1111_3344_amd import bssn as B
    du = B.to_device(I.smooth_random(G, seed=1))
    c = (ctypes.c_double * 3)(0.0, 0.0, 0.0)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    gp = ctypes.byref(B.c_grid(G))

    def best(nt, nph, lmax=4):
        work = torch.empty(2 * nt * (nph + 1) + 128 * (lmax + 1) ** 2,
                           dtype=torch.float64, device="cuda")
        out = torch.empty(2 * (lmax + 1) ** 2, dtype=torch.float64,
                          device="cuda")
        t = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            assert B.lib().bssn_multipole(
                gp, B.ptr(G, du), None, c, 0.5, 0, lmax, nt, nph,
                ctypes.c_void_p(work.data_ptr()),
                ctypes.c_void_p(out.data_ptr()), stream) == 0
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    # 16 times the points and the nodes: not far from 16 times the time (75
    # times when every point ran its own Newton iteration)
    print("[multipole] cost per point", flush=True)
    assert best(1024, 4096) <= 28 * best(64, 4096)
