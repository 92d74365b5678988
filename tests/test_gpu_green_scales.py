"""Row scales of the 16-bit Green's functions from tables, rows of one workgroup and of several."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# a row's largest A and 1/A over its valid entries set the powers of two; rows without a valid
# entry (and entries that are not positive) count for nothing
@pytest.mark.parametrize("nm", [1, 300, 16384, 16385, 40000])
@pytest.mark.parametrize("prec", ["RB_BF16", "RB_F16", "RB_F16X"])
def test_row_scales(nm, prec):
    from paper_2211_00316_amd import _lib

    n, omega, c0 = 5, 2.0 * math.pi * 4e5, 1500.0
    rng = np.random.default_rng(nm)
    A = np.exp(rng.uniform(-8.0, 3.0, (n, nm))).astype(np.float32)
    flags = np.where(rng.random((n, nm)) < 0.9, 0x80, 0).astype(np.uint8)
    flags[:, nm - 1] = 0x80          # the last node of a row is valid and its largest
    A[:, nm - 1] = np.float32(70.0) * 3.0 ** np.arange(n)
    flags[2] = 0
    A[4, 0] = 0.0
    tb = _lib.Tables.empty(n, nm, "cuda:0")
    for t in (tb.T, tb.rx_T, tb.rx_A, tb.rx_flags):
        t.zero_()
    tb.ux.fill_(1.0)
    tb.uy.zero_()
    tb.A.copy_(torch.from_numpy(A))
    tb.flags.copy_(torch.from_numpy(flags))
    gr = _lib.Context("cuda:0").build_green(tb, omega, c0,
                                            prec=getattr(_lib, prec))
    sk = np.float32(math.sqrt(omega / c0))

    def pow2(bound):
        return 2.0 ** (14 - math.frexp(float(bound))[1]) if bound > 0 else 1.0

    for e in range(n):
        a = A[e][(flags[e] & 0x80 != 0) & (A[e] > 0)]
        want = [pow2(a.max() * (np.float32(1) / sk)), pow2(np.float32(math.pi) * sk / a.min())] \
            if a.size else [1.0, 1.0]
        assert [float(gr.scales[0, e]), float(gr.scales[1, e])] == want
