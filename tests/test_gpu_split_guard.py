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
