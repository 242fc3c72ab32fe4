"""GPU check of the control words of the triangular solves spread over
workgroups (ticket, done count and published block counts: words 16, 17 and
32-63 of a workspace's control block): the last workgroup leaves them zero, as
the next solve on the same words expects.  The refinement runs two solves per
correction on one set of words that nothing else clears, so its iteration
count and convergence are asserted too: the FP32 solution of a well
conditioned problem has a backward error near 1e-7, above the tolerance of
1e-12, and each correction lowers it by orders of magnitude.
"""
import numpy as np
import pytest

from paper_1110_1553_amd import inputs

pytestmark = pytest.mark.gpu
WORDS = [16, 17] + list(range(32, 64))


def dev(X):
    import torch

    import paper_1110_1553_amd as h

    return h.colmajor(torch.from_numpy(np.ascontiguousarray(X)).cuda())


def solve_words(buf):
    """The words of the control block at the start of a workspace."""
    import torch

    torch.cuda.synchronize()
    return buf[:256].cpu().numpy().view(np.int32)[WORDS]


@pytest.mark.parametrize("nb,N,nrhs", [(64, 64, 1), (64, 449, 32), (256, 577, 5)])
def test_words_after_solves(hqr_lib, cuda, nb, N, nrhs):
    import paper_1110_1553_amd as h

    params = h.make_params(nb=nb, p=1, a=2, low="greedy")
    M = N + nb + 9
    print("nb %d %dx%d nrhs %d" % (nb, M, N, nrhs), flush=True)
    A, B = inputs.gaussian(M, N, 65), inputs.gaussian(M, nrhs, 66)
    work = h.lstsq(dev(A), dev(B), params)
    assert not solve_words(work.buf).any()
    bwork = h.ApplyWorkspace(M, nrhs, params)
    h.solve(dev(B), M, N, params, work, bwork=bwork)
    assert not solve_words(bwork.buf).any()


@pytest.mark.parametrize("nb,N", [(64, 449), (256, 300)])
def test_words_after_corrections(hqr_lib, cuda, nb, N):
    import torch

    import paper_1110_1553_amd as h
    from paper_1110_1553_amd import _lib

    M = 3 * N + 11
    params = h.make_params(nb=nb, p=1, a=2, low="greedy", precision="fp32")
    print("refinement nb %d %dx%d" % (nb, M, N), flush=True)
    A, b = dev(inputs.gaussian(M, N, 67)), dev(inputs.gaussian(M, 1, 68))
    x = torch.empty(N, dtype=torch.float64, device="cuda")
    nbytes = _lib.lstsq_ir_workspace_size(M, N, params)
    work = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    info = _lib.lstsq_ir_ptr(A.data_ptr(), M, N, M, b.data_ptr(), x.data_ptr(), 0, params, None, 30, 1e-12,
                             work.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream)
    assert info.converged and info.iterations >= 2
    assert not solve_words(work).any()
