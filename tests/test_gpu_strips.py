"""GPU parity of updates whose chunk holds one, two, three or four live strips
of 16 columns (the update kernels take one or two strips by rows, more one per
wave): right-hand-side counts on both sides of each limit, a matrix whose last
tile column has 5 or 21 columns, and every tile size.

The least-squares solution is compared with the oracle's, and Q^T B with the
identities R^T (Q^T B)(0:N) = A^T B and Q Q^T B = B; these matrices are well
conditioned (iid N(0,1), M >= 2N), so errors are a few hundred u (u = 1.1e-16)
and the bar is the 1e-12 of the other parity tests.
"""
import numpy as np
import pytest

from oracle import qr as oq
from paper_1110_1553_amd import inputs

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.mark.parametrize("nrhs", [1, 16, 17, 32, 33, 64, 81])
@pytest.mark.parametrize("nb,extra,a,low", [(64, 5, 65535, "flat"), (128, 21, 1, "binary"), (256, 5, 2, "greedy")])
def test_live_strips(hqr_lib, cuda, nb, extra, a, low, nrhs):
    import torch

    import paper_1110_1553_amd as h

    M, N = 5 * nb + 37, nb + extra
    params = h.make_params(nb=nb, p=1, a=a, low=low)
    ex = h.make_exec(spin_limit=4000000)
    A, B = inputs.gaussian(M, N, 41), inputs.gaussian(M, nrhs, 42)
    print("case nb %d %s %dx%d nrhs %d" % (nb, low, M, N, nrhs), flush=True)

    def dev(X):
        return h.colmajor(torch.from_numpy(np.ascontiguousarray(X)).cuda())

    dA, dB = dev(A), dev(B)
    h.lstsq(dA, dB, params, ex)
    x, ref = dB[:N].cpu().numpy(), oq.lstsq(A, B)
    assert np.linalg.norm(x - ref) <= TOL * np.linalg.norm(ref)

    dA, dB = dev(A), dev(B)
    work = h.factor(dA, params, ex)
    R = h.r_of(dA)
    h.apply_qt(dB, M, N, params, work, ex)
    top = dB[:N].cpu().numpy()
    assert np.linalg.norm(R.T @ top - A.T @ B) <= TOL * np.linalg.norm(A) * np.linalg.norm(B)
    h.apply_q(dB, M, N, params, work, ex)
    assert np.linalg.norm(dB.cpu().numpy() - B) <= TOL * np.linalg.norm(B)
