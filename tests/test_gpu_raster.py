"""The smallest-key pass of folded fans against the oracle where its segments of 64 runs and their
boxes of 16 have edges: fewer than 64 ray pairs (several rows of runs in a segment), exactly 64,
one more, segments that end inside a row, and a grid so fine that a box is taller than its height
field holds and that the lists of quads overflow (every quad there holds nodes; without the quads
that are then rasterised on the spot 4 % of the nodes differ).

Tolerances: the travel time and amplitude bounds of the parity tests (FP32 fields along a ray and
in a triangle; 1e-5 and 1e-4), on the nodes where both sides kept the same arrival; where two
arrivals are closer than the FP32 rounding of the residual either may be kept, 1e-3 of the nodes at
most, and coverage is decided by FP32 edge tests, 1e-4 of the nodes at most.
"""
import math

import numpy as np
import pytest

import phantoms as ph
from gpu_cases import C0, oracle_tables_of, rel_l2
from oracle.medium import Grid, Ring
from oracle.step import StepSetup
from oracle.trace import trace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, R, dx, rays", [(5, 0.02, 0.4e-3, 33), (4, 0.02, 0.4e-3, 65),
                                            (3, 0.02, 0.4e-3, 66), (4, 0.02, 0.4e-3, 150),
                                            (3, 0.01, 0.03e-3, 40)])
def test_folded_fans_at_segment_edges(n, R, dx, rays):
    import torch
    from paper_2211_00316_amd import _lib

    ds = 0.2e-3
    nx = int(math.ceil(2 * (R + 1e-3) / dx)) + 1
    x0 = -(nx - 1) * dx / 2
    st = StepSetup(Grid(nx, nx, dx, x0, x0, 0.9 * R), Ring(n, R), rays, ds,
                   int(math.ceil(2.5 * R / ds)) + 2)
    c = ph.gaussian_inclusion(nx, nx, dx, x0, x0, seed=14, amp=-300.0, sigma=0.15 * R,
                              centre_radius=0.3 * R, mask_radius=0.9 * R)
    tb_o, ns = oracle_tables_of(st, C0 / c)
    rays_o = trace(ns, st.grid, st.ring, st.n_rays, st.ds, st.max_steps, c0=st.c0)
    grid = _lib.Grid(nx, nx, dx, x0, x0, 0.9 * R)
    ring = _lib.Ring(n, R, 0.0)
    tp = _lib.TraceParams(rays, st.max_steps, ds, C0)
    cx = _lib.Context("cuda:0")
    print(f"folded fans n={n} rays={rays} grid={nx}", flush=True)
    tb = cx.trace_rays(grid, ring, tp,
                       torch.as_tensor(ns.astype(np.float32), device="cuda:0").contiguous())
    torch.cuda.synchronize()
    T, A = tb.T.cpu().numpy(), tb.A.cpu().numpy()
    flags = tb.flags.cpu().numpy()
    cx.close()
    valid = (flags & 0x80) != 0
    assert np.any(rays_o.K > 0)  # the fans do fold
    assert np.count_nonzero(valid != tb_o.valid) <= 1e-4 * valid.size
    both = valid & tb_o.valid
    same = both & (np.abs(T - tb_o.T) <= 1e-6 * tb_o.T)
    assert np.count_nonzero(both & ~same) <= 1e-3 * np.count_nonzero(both)
    assert rel_l2(T[same], tb_o.T[same]) <= 1e-5
    assert rel_l2(A[same], tb_o.A[same]) <= 1e-4
