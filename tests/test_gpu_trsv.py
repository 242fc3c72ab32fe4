"""GPU check of the triangular solves spread over workgroups (one per block of
64 unknowns and column, up to 32 columns) at the edges of blocks, tiles and
column counts.

The batched launch solves each column with a single workgroup that sums in the
same order, so the solutions must agree bit for bit; a second solve with the
same workspace must repeat the first (the control words are as they were
found).  The refined solutions of the mixed-precision path, which also solves
with R^T, are compared with the oracle's: iid N(0,1) with M >= 3 N, errors of
a few hundred u, bar 1e-12.
"""
import numpy as np
import pytest

from oracle import qr as oq
from paper_1110_1553_amd import inputs

pytestmark = pytest.mark.gpu


def dev(X):
    import torch

    import paper_1110_1553_amd as h

    return h.colmajor(torch.from_numpy(np.ascontiguousarray(X)).cuda())


@pytest.mark.parametrize("nb,N", [(64, 1), (64, 64), (64, 65), (64, 449), (128, 130), (256, 255), (256, 577)])
def test_blocks_and_columns(hqr_lib, cuda, nb, N):
    import torch

    import paper_1110_1553_amd as h

    params = h.make_params(nb=nb, p=1, a=2, low="greedy")
    ex = h.make_exec(spin_limit=4000000)
    M = N + nb + 9
    A = inputs.gaussian(M, N, 61)
    for nrhs in (1, 2, 32, 33):
        print("nb %d %dx%d nrhs %d" % (nb, M, N, nrhs), flush=True)
        B = inputs.gaussian(M, nrhs, 62)
        dA, dB, eA, eB = dev(A), dev(B), dev(A), dev(B)
        work = h.lstsq(dA, dB, params, ex)
        h.lstsq_batched([eA], [eB], params, ex)
        assert torch.equal(dB, eB)
        if nrhs == 2:
            bwork = h.ApplyWorkspace(M, nrhs, params)
            first, again = dev(B), dev(B)
            work = h.factor(dev(A), params, ex)
            h.solve(first, M, N, params, work, ex, bwork=bwork)
            h.solve(again, M, N, params, work, ex, bwork=bwork)
            assert torch.equal(first, again)


@pytest.mark.parametrize("nb,N", [(64, 65), (128, 449), (256, 300)])
def test_refinement(hqr_lib, cuda, nb, N):
    import paper_1110_1553_amd as h

    M = 3 * N + 11
    print("refinement nb %d %dx%d" % (nb, M, N), flush=True)
    A, b = inputs.gaussian(M, N, 63), inputs.gaussian(M, 1, 64)
    x = h.lstsq_ir(dev(A), dev(b).reshape(-1).contiguous(), h.make_params(nb=nb, p=1, a=2, low="greedy", precision="fp32"))[0]
    ref = oq.lstsq(A, b).reshape(-1)
    err = np.linalg.norm(x.cpu().numpy().reshape(-1) - ref) / np.linalg.norm(ref)
    print("  x %.2e" % err, flush=True)
    assert err <= 1e-12
