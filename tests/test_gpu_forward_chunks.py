"""Born forwards with given numbers of K chunks, fewer and more than the device's 8 XCDs."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


# FP32 takes K chunks as the tuning gives them; with node weights the 16-bit types use the same
# kernel. Products of FP32 values: 3 x 2^-24 each and the sum's roundings; 16-bit: G v rounded once
# more (2^-9, 2^-12, of random sign), G exact.
@pytest.mark.parametrize("n, nm, chunks", [(300, 1000, 1), (300, 1000, 3), (300, 1000, 7),
                                           (300, 1000, 8), (300, 1000, 9), (130, 100, 5)])
@pytest.mark.parametrize("prec", ["RB_F32", "RB_BF16", "RB_F16"])
def test_chunks(n, nm, chunks, prec):
    from paper_2211_00316_amd import _lib

    g = torch.Generator(device="cuda:0").manual_seed(n + chunks)
    dt = {"RB_F32": torch.float32, "RB_BF16": torch.bfloat16, "RB_F16": torch.float16}[prec]
    vals = torch.randn(2, n, nm, generator=g, device="cuda:0").to(dt)
    w = torch.view_as_complex(torch.randn(nm, 2, generator=g, device="cuda:0"))
    delta = torch.rand(nm, generator=g, device="cuda:0")
    p = getattr(_lib, prec)
    if prec == "RB_F32":
        G = torch.complex(vals[0], vals[1])
        gr = _lib.Green(G, G, p)
    else:
        n_pad, m_pad = (n + 31) // 32 * 32, (nm + 31) // 32 * 32
        G = torch.zeros(2, n, m_pad, dtype=dt, device="cuda:0")
        G[:, :, :nm] = vals
        gr = _lib.Green(G, torch.zeros(3, 2, nm, n_pad, dtype=dt, device="cuda:0"), p,
                        torch.ones(2, n, device="cuda:0"))
    ctx = _lib.Context("cuda:0")
    ctx.set_tuning({"n": n, "n_mask": nm, "prec": p, "fwd_tile": 1, "fwd_splitk": chunks,
                    "fwd_ms": 1.0})
    d = ctx.born_forward(gr, w, delta)
    X = torch.complex(vals[0].double(), vals[1].double())
    ref = (X * (w.to(torch.complex128) * delta.double())) @ X.t().contiguous()
    assert torch.equal(d, d.t())
    err = torch.linalg.norm(torch.view_as_real(d.to(torch.complex128) - ref))
    bound = 2.0 * (3.0 + math.sqrt(nm)) * 2.0 ** -24 + 6 * 2.0 ** -24
    bound += {"RB_F32": 0.0, "RB_BF16": 2.0 ** -9, "RB_F16": 2.0 ** -12}[prec]
    assert float(err / torch.linalg.norm(torch.view_as_real(ref))) <= bound
