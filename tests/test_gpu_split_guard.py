"""Which FP32 contractions run on split operands and what those keep: the FP32 kernels that follow
them give other last bits, so a call whose results equal, bit for bit, those of the same call with
an infinity planted in a column of no interest was turned down.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

OMEGA, D_OMEGA = 2 * math.pi * 300e3, 2 * math.pi * 30e3


def randc(g, *shape):
    return torch.view_as_complex(torch.randn(*shape, 2, generator=g, device="cuda:0"))


@pytest.fixture(scope="module")
def ctx():
    from paper_2211_00316_amd import _lib

    return _lib.Context("cuda:0")


def backproject(ctx, H, R):
    from paper_2211_00316_amd import _lib

    c = torch.full((H.shape[2],), 1500.0, device="cuda:0", dtype=torch.float64)
    return ctx.backproject(_lib.Green(torch.zeros_like(H[0]), H, _lib.RB_F32), R, c, OMEGA,
                           D_OMEGA)


# small: a few entries of the last row far below its others. With 257 and 513 transducers that row
# is a row slab of its own.
@pytest.mark.parametrize("n", [70, 256, 257, 513])
@pytest.mark.parametrize("small", [False, True])
def test_backproject_runs_split(ctx, n, small):
    g = torch.Generator(device="cuda:0").manual_seed(n)
    H = torch.stack([randc(g, n, 640) for _ in range(3)]).contiguous()
    R = randc(g, n, n)
    if small:
        H[:, n - 1, 300:305] *= 2.0 ** -12
    dm = backproject(ctx, H, R)
    H[0, 0, 0] = complex(math.inf, 0.0)
    plain = backproject(ctx, H, R)
    assert not torch.isfinite(plain[0]) and torch.isfinite(plain[1:]).all()
    assert not torch.equal(dm[1:], plain[1:])


def rel(a, b):
    return float(torch.linalg.norm(a.double() - b.double()) / torch.linalg.norm(b.double()))


# A node's result keeps FP32's accuracy whatever else its column, its rows or R hold. dead: the
# transducers with the large entries of the nodes looked at have no data, and what is left lies
# 2^-18 (2^-40) below its rows' other nodes. outlier: one residual is 1e12 times the others,
# between transducers that do not see the nodes looked at. K products of (3 x 2^-24) each and their
# sum's roundings, as in the comparison with FP64 of the other operands.
@pytest.mark.parametrize("case", ["dead18", "dead40", "outlier"])
def test_backproject_keeps_small_entries(ctx, case):
    n, nm, part = 70, 600, slice(100, 200)
    g = torch.Generator(device="cuda:0").manual_seed(9)
    H = torch.stack([randc(g, n, nm) for _ in range(3)]).contiguous()
    R = randc(g, n, n)
    if case == "outlier":
        R[3, 9] = 1e12
        H[:, [3, 9], part] = 0
    else:
        R[:35] = 0
        R[:, :35] = 0
        H[:, 35:, part] *= 2.0 ** -int(case[4:])
    dm = backproject(ctx, H, R)[part]
    Hd, Rd = H[:, :, part].to(torch.complex128), R.to(torch.complex128)
    acc = sum((x * (Rd @ x)).sum(0) for x in Hd).real
    ref = -2.0 * D_OMEGA / ((2.0 * math.pi) ** 3 * OMEGA * 1500.0 ** 2) * acc
    assert rel(dm, ref) <= 2.0 * (3.0 + math.sqrt(n)) * 2.0 ** -24 * math.sqrt(3.0)


# Values below 2^-100, whose last part FP32's exponents might not hold, go to the FP32 kernels (and
# the smallest that do not run split). R is large enough for results in FP32's normal range.
@pytest.mark.parametrize("exponent, split", [(-104, False), (-90, True)])
def test_adjoint_of_tiny_entries(ctx, exponent, split):
    from paper_2211_00316_amd import _lib

    n, nm, part = 70, 600, slice(100, 200)
    g = torch.Generator(device="cuda:0").manual_seed(11)
    unit = torch.polar(1.0 + torch.rand(n, nm, generator=g, device="cuda:0"),
                       math.pi / 4 + 0.5 * torch.rand(n, nm, generator=g, device="cuda:0"))
    G = unit.clone()
    G[:, part] *= 2.0 ** exponent
    R = randc(g, n, n) * 2.0 ** 100
    w = torch.ones(nm, dtype=torch.complex64, device="cuda:0")
    out = ctx.born_adjoint(_lib.Green(G, G, _lib.RB_F32), w, R)
    X = G.to(torch.complex128).conj().resolve_conj()
    ref = (X * (R.to(torch.complex128) @ X)).sum(0).real
    assert rel(out[part], ref[part]) <= 2.0 * (3.0 + math.sqrt(n)) * 2.0 ** -24 * math.sqrt(2.0)
    G[0, 0] = complex(math.inf, 0.0)
    plain = ctx.born_adjoint(_lib.Green(G, G, _lib.RB_F32), w, R)
    assert torch.equal(out[1:], plain[1:]) != split


def forward(ctx, G, delta):
    from paper_2211_00316_amd import _lib

    w = torch.ones(G.shape[1], dtype=torch.complex64, device="cuda:0")
    return ctx.born_forward(_lib.Green(G, G, _lib.RB_F32), w, delta)


# Every pair of transducers keeps FP32's accuracy. The first 35 and the others each see a node of
# their own; what one of each see together are 100 nodes where both are 2^-16 (2^-40) of their
# rows' others. gauss: a perturbation that falls off to FP32's smallest numbers, which must not
# cost the second pass. K products of (3 x 2^-24) and the roundings of their sum, as in the
# comparison with FP64 of the other operands, and those of G v.
@pytest.mark.parametrize("case", ["cross16", "cross40", "gauss"])
def test_forward_keeps_small_entries(ctx, case):
    n, nm = 70, 20000
    g = torch.Generator(device="cuda:0").manual_seed(6)
    G = randc(g, n, nm)
    delta = torch.zeros(nm, device="cuda:0")
    if case == "gauss":
        x = torch.linspace(-16.0, 16.0, nm, device="cuda:0", dtype=torch.float64)
        delta = (1e-9 * torch.exp(-0.5 * x * x)).float()
        assert (delta == 0).any() and ((delta > 0) & (delta < 1e-40)).any()
    else:
        G[:, 100:200] *= 2.0 ** -int(case[5:])
        G[:35, 778] = 0
        G[35:, 777] = 0
        delta[100:200] = 1.0
        delta[777:779] = 1.0
    d = forward(ctx, G, delta)
    X = G.to(torch.complex128)
    ref = (X * delta.double()) @ X.t().contiguous()
    pairs = slice(None) if case == "gauss" else slice(35, None)
    K = int((delta != 0).sum())
    err = rel(torch.view_as_real(d[:35, pairs]), torch.view_as_real(ref[:35, pairs]))
    assert err <= 2.0 * (3.0 + math.sqrt(K)) * 2.0 ** -24 + 6 * 2.0 ** -24
    G[0, 0] = complex(math.inf, 0.0)
    assert not torch.equal(d[1:, 1:], forward(ctx, G, delta)[1:, 1:])


# A call that the split form turns down pays for little more than the FP32 kernel. That issues 16/6
# of the split kernel's MFMA time per product and 1.18 times its products (R's triangle in blocks
# of 256 rows instead of 64), 3.14 together; the infinity is met in the first columns. A fifth of
# that is left for what the MFMAs do not bound.
def test_backproject_turned_down_time(ctx):
    from paper_2211_00316_amd import _lib

    n, nm = 1024, 40000
    g = torch.Generator(device="cuda:0").manual_seed(4)
    H = torch.stack([randc(g, n, nm) for _ in range(3)]).contiguous()
    R = randc(g, n, n)
    c = torch.full((nm,), 1500.0, device="cuda:0", dtype=torch.float64)
    gr = _lib.Green(torch.zeros_like(H[0]), H, _lib.RB_F32)

    def best():
        times = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            ctx.backproject(gr, R, c, OMEGA, D_OMEGA)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times[1:])

    split = best()
    H[0, 0, 0] = complex(math.inf, 0.0)
    down = best()
    print(f"split {split:.2f} ms, turned down {down:.2f} ms")
    assert down <= 1.2 * 3.14 * split


# Calls of which a CU's column blocks (64 nodes) take three steps of 16 transducers, over all
# components, run on the FP32 kernel alone, longer ones split.
@pytest.mark.parametrize("kind, n, nm, split", [
    ("backproject", 16, 500, False), ("backproject", 17, 500, True),
    ("backproject", 16, 40000, True), ("adjoint", 48, 500, False), ("adjoint", 49, 500, True),
    ("adjoint", 16, 40000, False), ("adjoint", 17, 40000, True), ("adjoint", 8, 70000, True)])
def test_short_calls_run_on_fp32_kernels(ctx, kind, n, nm, split):
    from paper_2211_00316_amd import _lib

    g = torch.Generator(device="cuda:0").manual_seed(n)
    H = torch.stack([randc(g, n, nm) for _ in range(3)]).contiguous()
    R = randc(g, n, n)
    w = torch.ones(nm, dtype=torch.complex64, device="cuda:0")

    def call():
        if kind == "backproject":
            return backproject(ctx, H, R)
        return ctx.born_adjoint(_lib.Green(H[0].contiguous(), H, _lib.RB_F32), w, R)

    out = call()
    H[0, 0, 0] = complex(math.inf, 0.0)
    assert torch.equal(out[1:], call()[1:]) != split


# Forwards over few nodes run on the FP32 kernel alone (large rings up to 160 nodes), others split.
@pytest.mark.parametrize("n, nm, split", [(70, 32, False), (70, 33, True), (1024, 33, True),
                                          (1025, 160, False), (1025, 161, True)])
@pytest.mark.parametrize("weights", [True, False])
def test_short_forwards_run_on_fp32_kernels(ctx, n, nm, split, weights):
    from paper_2211_00316_amd import _lib

    g = torch.Generator(device="cuda:0").manual_seed(n + nm)
    G = randc(g, n, nm)
    w = randc(g, nm) if weights else None
    delta = torch.randn(nm, generator=g, device="cuda:0") if weights else None
    d = ctx.born_forward(_lib.Green(G, G, _lib.RB_F32), w, delta)
    X = G.to(torch.complex128)
    v = w.to(torch.complex128) * delta.double() if weights else 1.0
    ref = (X * v) @ X.t().contiguous()
    # K products of (3 x 2^-24), their sum's roundings and those of w delta and G v
    err = rel(torch.view_as_real(d), torch.view_as_real(ref))
    assert err <= 2.0 * (3.0 + math.sqrt(nm)) * 2.0 ** -24 + 6 * 2.0 ** -24
    G[0, 0] = complex(math.inf, 0.0)
    plain = ctx.born_forward(_lib.Green(G, G, _lib.RB_F32), w, delta)
    assert torch.equal(d[1:, 1:], plain[1:, 1:]) != split
