"""The FP32 contractions on split FP16 operands against FP64 sums, and the calls that the split
form hands to the FP32 kernels: infinities, values past FP16's range, columns or rows far below
the others.

Tolerance: a product carries at most 3 x 2^-24 (two representations and the dropped lo lo'), a sum
of K terms of random phase a rounding walk of about sqrt(K) 2^-24 relative to its rms; twice the
sum of both bounds the relative 2-norm over results whose terms do not cancel.
"""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

OMEGA, D_OMEGA = 2 * math.pi * 300e3, 2 * math.pi * 30e3


def tol(K):
    return 2.0 * (3.0 + math.sqrt(K)) * 2.0 ** -24


def randc(g, *shape):
    z = torch.randn(*shape, 2, generator=g, device="cuda:0", dtype=torch.float32)
    return torch.view_as_complex(z)


def direction(H, R, c, n_comp=3):
    """-S Re sum H (R H) in complex128, S of the lossless back-projection."""
    H, R = H.to(torch.complex128), R.to(torch.complex128)
    acc = sum((H[k] * (R @ H[k])).sum(0) for k in range(n_comp))
    S = 2 * D_OMEGA / ((2 * math.pi) ** 3 * OMEGA * c ** 2)
    return -(S * acc.real)


def rel(a, b):
    a, b = a.double(), b.double()
    return float(torch.linalg.norm(a - b) / torch.linalg.norm(b))


@pytest.fixture(scope="module")
def ctx():
    from paper_2211_00316_amd import _lib

    return _lib.Context("cuda:0")


# one transducer tile, partial tiles and slabs, an odd number of slabs; node tiles of 128 with
# remainders; the K tails of the pipelined loop (1 to 6 steps of 16 and more)
@pytest.mark.parametrize("n, nm", [(3, 1), (16, 130), (17, 127), (32, 128), (48, 257), (64, 1000),
                                   (80, 385), (96, 64), (255, 300), (256, 129), (257, 640),
                                   (300, 2500), (513, 700), (770, 200)])
def test_backproject_and_adjoint_match_fp64(ctx, n, nm):
    from paper_2211_00316_amd import _lib

    g = torch.Generator(device="cuda:0").manual_seed(n * 1000 + nm)
    amp = torch.exp(torch.randn(n, 1, generator=g, device="cuda:0"))   # rows of other sizes
    H = torch.stack([randc(g, n, nm) * amp * 1e-3 for _ in range(3)]).contiguous()
    G = (randc(g, n, nm) * amp * 30.0).contiguous()
    R = randc(g, n, n) * 1e-2
    c = 1500.0 + 30.0 * torch.rand(nm, generator=g, device="cuda:0", dtype=torch.float64)
    gr = _lib.Green(G, H, _lib.RB_F32)
    dm = ctx.backproject(gr, R, c, OMEGA, D_OMEGA)
    assert rel(dm, direction(H, R, c)) <= tol(n) * math.sqrt(3)
    w = randc(g, nm)
    out = ctx.born_adjoint(gr, w, R)
    X = G.to(torch.complex128).conj().resolve_conj()
    ref = (w.to(torch.complex128).conj() * (X * (R.to(torch.complex128) @ X)).sum(0)).real
    assert rel(out, ref) <= tol(n) * math.sqrt(2)
    noalloc = torch.empty_like(dm)
    ctx.backproject_noalloc(gr, R, c, OMEGA, D_OMEGA, noalloc)
    assert torch.equal(noalloc, dm)


@pytest.mark.parametrize("case", ["inf", "nan_r", "spike", "column", "row", "unsampled"])
def test_backproject_outside_the_split_range(ctx, case):
    from paper_2211_00316_amd import _lib

    n, nm = 70, 5000
    g = torch.Generator(device="cuda:0").manual_seed(5)
    H = torch.stack([randc(g, n, nm) for _ in range(3)]).contiguous()
    R = randc(g, n, n)
    c = torch.full((nm,), 1500.0, device="cuda:0", dtype=torch.float64)
    bad = torch.zeros(nm, dtype=torch.bool, device="cuda:0")
    if case == "inf":
        H[1, 7, 33] = complex(math.inf, 0.0)
        bad[33] = True
    elif case == "nan_r":
        R[3, 9] = complex(math.nan, 0.0)
        bad[:] = True
    elif case == "spike":       # past 65504 after the row's scale
        H[0, 11, 4000] = 3e6
    elif case == "column":      # a column far below the others keeps its relative accuracy
        H[:, :, 100:140] *= 1e-9
    elif case == "row":         # a row of the largest exponents
        H[:, 5] *= 1e15
        R[5] *= 1e-15
        R[:, 5] *= 1e-15
    elif case == "unsampled":   # nothing but a few columns is not zero
        keep = H[:, :, 2003:2007].clone()
        H.zero_()
        H[:, :, 2003:2007] = keep * 1e-6
    dm = ctx.backproject(_lib.Green(torch.zeros_like(H[0]), H, _lib.RB_F32), R, c, OMEGA, D_OMEGA)
    ref = direction(H, R, c)
    assert not torch.isfinite(dm[bad]).any()
    ok = ~bad
    if ok.any():
        assert torch.isfinite(dm[ok]).all()
        live = ok & (ref != 0)
        scale = ref[live].abs()
        if case == "column":
            part = torch.zeros_like(ok)
            part[100:140] = True
            assert rel(dm[part], ref[part]) <= tol(n) * math.sqrt(3)
        assert float(((dm[live].double() - ref[live]).abs() / scale).median()) <= tol(n) * 4
        assert rel(dm[ok], ref[ok]) <= tol(n) * math.sqrt(3)


def product(G, v):
    G = G.to(torch.complex128)
    return (G * v) @ G.t().contiguous()


# tile remainders, one to a few stages of 16 nodes and K chunks with a partial last stage
@pytest.mark.parametrize("n, nm", [(3, 1), (5, 3), (64, 17), (127, 64), (128, 1000), (129, 4100),
                                   (200, 333), (257, 9001)])
@pytest.mark.parametrize("weights", [True, False])
def test_forward_matches_fp64(ctx, n, nm, weights):
    from paper_2211_00316_amd import _lib

    g = torch.Generator(device="cuda:0").manual_seed(n * 7 + nm)
    amp = torch.exp(torch.randn(n, 1, generator=g, device="cuda:0"))
    G = (randc(g, n, nm) * amp * 0.03).contiguous()
    w = delta = None
    v = torch.ones(nm, dtype=torch.complex128, device="cuda:0")
    if weights:
        w = randc(g, nm) * 1e4
        delta = torch.randn(nm, generator=g, device="cuda:0") * 1e-9
        v = w.to(torch.complex128) * delta.double()
    d = ctx.born_forward(_lib.Green(G, G, _lib.RB_F32), w, delta)
    assert torch.equal(d, d.t())
    # the FP32 products w delta and G v add three roundings
    assert rel(torch.view_as_real(d), torch.view_as_real(product(G, v))) <= tol(nm) + 6 * 2.0 ** -24


@pytest.mark.parametrize("case", ["inf", "spike", "row", "point", "decades", "weight_inf"])
def test_forward_outside_the_split_range(ctx, case):
    from paper_2211_00316_amd import _lib

    n, nm = 70, 20000
    g = torch.Generator(device="cuda:0").manual_seed(6)
    G = randc(g, n, nm)
    w = torch.ones(nm, dtype=torch.complex64, device="cuda:0")
    delta = torch.randn(nm, generator=g, device="cuda:0")
    bad = torch.zeros(n, n, dtype=torch.bool, device="cuda:0")
    if case == "inf":
        G[7, 33] = complex(math.inf, 0.0)
        bad[7] = bad[:, 7] = True
    elif case == "spike":          # far past the rms of its row's sample
        G[11, 4001] = 3e7
    elif case == "row":            # a row whose sample is zero, and tiny elsewhere
        keep = G[5, 10001].clone()
        G[5] = 0
        G[5, 10001] = keep * 1e-9
    elif case == "point":          # a single scatterer
        delta.zero_()
        delta[777] = 2.5
    elif case == "decades":        # weights over many decades
        delta *= torch.exp(-30.0 * torch.rand(nm, generator=g, device="cuda:0"))
    elif case == "weight_inf":
        delta[3] = math.inf
        bad[:] = True
    d = ctx.born_forward(_lib.Green(G, G, _lib.RB_F32), w, delta)
    assert not torch.isfinite(torch.view_as_real(d[bad])).all(-1).any()
    ok = ~bad
    if ok.any():
        ref = product(G, w.to(torch.complex128) * delta.double())[ok]
        x = d[ok]
        assert torch.isfinite(torch.view_as_real(x)).all()
        assert rel(torch.view_as_real(x), torch.view_as_real(ref)) <= tol(nm) + 6 * 2.0 ** -24
        if case == "row":
            assert rel(torch.view_as_real(d[5]), torch.view_as_real(
                product(G, w.to(torch.complex128) * delta.double())[5])) <= tol(nm)
