"""GPU check of the copies between a column-major matrix and tiles.

Ragged sizes around the copies' 8-column pieces and the tiles, leading
dimensions beyond the row count, and right-hand-side counts around a 64-column
chunk.  The batch runs in a workspace full of NaN: padding that the copy in
leaves as it is must not reach a result, so R, V, the solutions and the
residual parts equal, bit for bit, the ones of each problem on its own (whose
copy fills all padding with zeros).  The rows below M must stay as they were.
R is compared with the oracle's too (well conditioned matrices: 1e-12).
"""
import numpy as np
import pytest

from oracle import qr as oq
from paper_1110_1553_amd import inputs

pytestmark = pytest.mark.gpu
MARK = -7.25


@pytest.mark.parametrize("nb", [64, 128, 256])
def test_batched_copies(hqr_lib, cuda, nb):
    import torch

    import paper_1110_1553_amd as h
    from paper_1110_1553_amd import _lib

    params = h.make_params(nb=nb, p=1, a=2, low="greedy")
    ex = h.make_exec(spin_limit=4000000)
    sizes = [(1, 1, 1), (9, 7, 2), (nb, nb, 1), (nb + 1, 8, 63), (2 * nb - 1, 9, 64), (3 * nb + 5, nb + 1, 65),
             (2 * nb + 33, nb - 1, 129), (nb + 77, 17, 0)]
    print("nb %d: %s" % (nb, sizes), flush=True)

    def padded(X, extra):
        buf = torch.full((max(X.shape[1], 1), X.shape[0] + extra), MARK, dtype=torch.float64, device="cuda")
        view = buf.t()[:X.shape[0], :X.shape[1]]
        view.copy_(torch.from_numpy(X))
        return buf, view

    host = [(inputs.gaussian(m, n, 50 + q), inputs.gaussian(m, max(r, 1), 80 + q)[:, :r])
            for q, (m, n, r) in enumerate(sizes)]
    As = [padded(A, q % 3) for q, (A, _) in enumerate(host)]
    Bs = [padded(B, (q + 1) % 3) for q, (_, B) in enumerate(host)]
    batch = _lib.Batch([m for m, _, _ in sizes], [n for _, n, _ in sizes], [r for _, _, r in sizes], params, ex)
    nbytes = batch.workspace_size()
    work = torch.full(((nbytes + 7) // 8,), float("nan"), dtype=torch.float64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    batch.bind([v.data_ptr() for _, v in As], [b.shape[1] for b, _ in As],
               [v.data_ptr() for _, v in Bs], [b.shape[1] for b, _ in Bs], work.data_ptr(), nbytes, stream)
    batch.run(work.data_ptr(), nbytes, stream)
    torch.cuda.synchronize()
    assert batch.status(work.data_ptr(), stream)[0] == 0
    for q, (m, n, r) in enumerate(sizes):
        A, B = host[q]
        dA = h.colmajor(torch.from_numpy(np.ascontiguousarray(A)).cuda())
        if r:
            dB = h.colmajor(torch.from_numpy(np.ascontiguousarray(B)).cuda())
            h.lstsq(dA, dB, params, ex)
            assert torch.equal(Bs[q][1], dB), (q, "B")
        else:
            h.factor(dA, params, ex)
        assert torch.equal(As[q][1], dA), (q, "A")
        for buf, _ in (As[q], Bs[q]):
            assert bool((buf[:, m:] == MARK).all()), (q, "rows below the matrix")
        R, ref = np.triu(As[q][1].cpu().numpy()[:n]), oq.r_of(oq.factor(A)[0])
        err = np.linalg.norm(np.abs(R) - np.abs(ref)) / np.linalg.norm(ref)
        print("  %s R %.2e" % (sizes[q], err), flush=True)
        assert err <= 1e-12
    batch.close()
