"""GPU parity of the panel column loop where it can go wrong: every row-slot
count of the three panel kinds (the tile sizes fix them), columns of very
different scale (each column's tail, head and dot products are formed from
the unscaled column), a zero column and a column that is zero below its head.

Householder QR of A D (D diagonal, positive) has R D, so R is compared column
by column, relative to the column: 1e-12 in FP64 as in the other parity
tests, 10 sqrt(MN) u_f in FP32 (u_f = 2^-24, the backward error of Householder
QR on these well-conditioned matrices).
"""
import numpy as np
import pytest

from oracle import qr as oq
from paper_1110_1553_amd import inputs

pytestmark = pytest.mark.gpu


def column_errors(R, Rref):
    a, b = oq.sign_normalize(R), oq.sign_normalize(Rref)
    n = np.linalg.norm(b, axis=0)
    return np.linalg.norm(a - b, axis=0) / np.where(n > 0, n, 1.0)


# M x N with all panels of a tile, one ragged tile column, and one column
SHAPES = [(600, 256), (530, 200), (257, 1)]


@pytest.mark.parametrize("dtype,scale", [("f64", 100.0), ("f32", 8.0)])
@pytest.mark.parametrize("a,low", [(65535, "flat"), (1, "binary")])
@pytest.mark.parametrize("nb", [64, 128, 256])
def test_column_scales(hqr_lib, cuda, nb, a, low, dtype, scale):
    import torch

    import paper_1110_1553_amd as h

    params = h.make_params(nb=nb, p=1, a=a, low=low)
    for M, N in SHAPES:
        A = inputs.gaussian(M, N, 31)
        # column scales 10^(-scale) .. 10^scale in no order
        A = A * 10.0 ** (scale * np.cos(1.7 * np.arange(N)))
        if N > 1:
            A[1:, 0] = 0.0   # zero below its head: the first reflector is the identity
            A[:, -1] = 0.0   # a zero column
        t = torch.float64 if dtype == "f64" else torch.float32
        dA = h.colmajor(torch.from_numpy(np.ascontiguousarray(A)).to(t).cuda())
        A = np.asfortranarray(dA.cpu().numpy().astype(np.float64))  # the oracle sees the rounded entries
        h.factor(dA, params, h.make_exec(spin_limit=4000000), timeout_s=60.0)
        R = h.r_of(dA).astype(np.float64)
        err = column_errors(R, oq.r_factor(A)).max()
        tol = 1e-12 if dtype == "f64" else 10.0 * np.sqrt(M * N) * 2.0 ** -24
        print("case %s nb %d %s %dx%d: column error %.3e" % (dtype, nb, low, M, N, err), flush=True)
        assert np.all(np.isfinite(R)) and err <= tol, (M, N, err)
