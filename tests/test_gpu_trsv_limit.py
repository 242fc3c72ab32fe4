"""GPU check that the caller's spin limit bounds the waits of the triangular
solves spread over workgroups.

One tile and 32 right-hand sides: the application of Q^T is a single task that
waits for nothing, and the solve has four blocks per column, each of which
polls while the one before it takes a 64-step substitution.  With a limit of one poll the
call must therefore report the watchdog (and end at once); with the default limit the same
workspaces then give the solution, as if nothing had happened.
"""
import numpy as np
import pytest

from oracle import qr as oq
from paper_1110_1553_amd import inputs

pytestmark = pytest.mark.gpu


def test_spin_limit_of_the_solve(hqr_lib, cuda):
    import torch

    import paper_1110_1553_amd as h
    from paper_1110_1553_amd import _lib

    n, nrhs = 256, 32
    params = h.make_params(nb=256, p=1, a=1, low="flat")
    A = inputs.gaussian(n, n, 71) + 20.0 * np.eye(n)  # well conditioned
    B = inputs.gaussian(n, nrhs, 72)

    def dev(X):
        return h.colmajor(torch.from_numpy(np.ascontiguousarray(X)).cuda())

    work = h.factor(dev(A), params)
    bwork = h.ApplyWorkspace(n, nrhs, params)
    print("solve %dx%d with %d columns, spin limit 1" % (n, n, nrhs), flush=True)
    with pytest.raises(_lib.HQRError) as e:
        h.solve(dev(B), n, n, params, work, h.make_exec(spin_limit=1), bwork=bwork)
    assert e.value.code == 2
    X = dev(B)
    h.solve(X, n, n, params, work, bwork=bwork)
    ref = oq.lstsq(A, B)
    assert np.linalg.norm(X.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)
