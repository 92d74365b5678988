"""The two forms of the ray tracer, chosen by the wavefronts of a launch: coefficients in LDS where
the card is full, loaded a step ahead into registers where it is not. The forms differ in when they
load, not in any operation, so tables traced in one launch (the first form) and in chunks of few
transducers (the second) are equal in every bit; ragged last groups of rays and chunks included.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, rays, part, lossy", [(96, 1100, 40, False), (97, 2047, 7, False),
                                                  (256, 961, 90, True), (130, 2048, 1, True)])
def test_forms_agree_bitwise(n, rays, part, lossy):
    from paper_2211_00316_amd import _lib

    R, dx, nx, ds, c0 = 8e-3, 0.4e-3, 48, 0.2e-3, 1500.0
    x0 = -0.5 * (nx - 1) * dx
    grid = _lib.Grid(nx, nx, dx, x0, x0, 0.7 * R)
    ring = _lib.Ring(n, R, 0.1)
    tp = _lib.TraceParams(rays, int(math.ceil(2.5 * R / ds)) + 2, ds, c0)
    ax = x0 + dx * torch.arange(nx, device="cuda:0")
    y, x = torch.meshgrid(ax, ax, indexing="ij")
    ns = (1.0 + 0.08 * torch.exp(-((x - 1e-3) ** 2 + y ** 2) / (2 * (1.2e-3) ** 2))).float()
    aw = (5.0 + 20.0 * (x > 0)).float().contiguous()
    ns = ns.contiguous()
    n_mask = int((x * x + y * y <= (0.7 * R) ** 2).sum())
    per = (tp.max_steps + 1) * rays * 25 + n_mask * 8 + rays * 32
    out = []
    for budget in (1 << 32, per * part + per // 2):
        cx = _lib.Context("cuda:0")
        cx.set_sample_budget(budget)
        print(f"trace forms n={n} rays={rays} lossy={lossy} budget={budget}", flush=True)
        out.append(cx.trace_rays_lossy(grid, ring, tp, ns, aw) if lossy
                   else cx.trace_rays(grid, ring, tp, ns))
        torch.cuda.synchronize()
        cx.close()
    a, b = out
    assert bool(((a.flags & 0x80) != 0).any())
    for name in ("T", "A", "ux", "uy", "flags", "rx_T", "rx_A", "rx_flags"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
