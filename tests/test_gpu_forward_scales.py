"""16-bit Born forward with node weights and row scales whose powers of two cancel only together."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# G near 2^-27 under row scales of 2^40, weights of 2^100 (and the reverse): the result lies well
# inside FP32, a product with one of the factors alone does not. Operands are exact in both types
# (sums of 200 products of 5 bits), so only FP32 additions round: 200 x 2^-24.
@pytest.mark.parametrize("prec", ["RB_BF16", "RB_F16"])
@pytest.mark.parametrize("row, weight", [(40, 100), (-40, -100)])
def test_weights_and_row_scales(prec, row, weight):
    from paper_2211_00316_amd import _lib

    n, nm = 40, 200
    dt = torch.bfloat16 if prec == "RB_BF16" else torch.float16
    g = torch.Generator(device="cuda:0").manual_seed(2)
    n_pad, m_pad = (n + 31) // 32 * 32, (nm + 31) // 32 * 32
    G = torch.zeros(2, n, m_pad, dtype=dt, device="cuda:0")
    vals = torch.randint(-16, 17, (2, n, nm), generator=g, device="cuda:0").double() * 2.0 ** 9
    G[:, :, :nm] = vals.to(dt)
    scales = torch.full((2, n), 2.0 ** row, device="cuda:0")
    H = torch.zeros(3, 2, nm, n_pad, dtype=dt, device="cuda:0")
    w = torch.full((nm,), 2.0 ** weight, dtype=torch.complex64, device="cuda:0")
    ctx = _lib.Context("cuda:0")
    d = ctx.born_forward(_lib.Green(G, H, getattr(_lib, prec), scales), w,
                         torch.ones(nm, device="cuda:0"))
    X = torch.complex(vals[0], vals[1]) * 2.0 ** -row
    ref = (X * 2.0 ** weight) @ X.t().contiguous()
    assert torch.isfinite(torch.view_as_real(d)).all()
    err = torch.linalg.norm(torch.view_as_real(d.to(torch.complex128) - ref))
    assert float(err / torch.linalg.norm(torch.view_as_real(ref))) <= 200 * 2.0 ** -24
