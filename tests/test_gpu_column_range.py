"""GPU parity of the panel column loop at the ends of its range: products of
raw columns that overflow or underflow while every norm does not.

A = G D with D diagonal, powers of two, so that R(A) = R(G) D: the columns of A
are near the magnitude where the square of a norm still is representable, and
the last one, parallel to the first (so that what is left of it below its
diagonal is rounding), is larger or smaller still.  Its product with the first
one's tail is outside the range of the type.  R is compared column by column
relative to the column: 1e-12 in FP64, 10 sqrt(MN) u_f in FP32, as for
moderate columns.  These twelve columns are the first panel, or a later one of a
block whose other panels are moderate.

An identity reflector (a column that is zero below its head) leaves the other
columns as they are, also one that holds an infinity.
"""
import numpy as np
import pytest

from oracle import qr as oq
from paper_1110_1553_amd import inputs

pytestmark = pytest.mark.gpu
TYPES = {"f64": ([(498, 548), (-498, -565)], 1e-12), "f32": ([(56, 73), (-56, -92)], None)}


def run(A, dtype, params):
    import torch

    import paper_1110_1553_amd as h

    t = torch.float64 if dtype == "f64" else torch.float32
    dA = h.colmajor(torch.from_numpy(np.ascontiguousarray(A)).to(t).cuda())
    h.factor(dA, params, h.make_exec(spin_limit=4000000))
    return h.r_of(dA).astype(np.float64)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("a,low", [(65535, "flat"), (1, "binary")])
@pytest.mark.parametrize("nb,first", [(64, 0), (64, 32), (128, 0), (128, 96), (256, 0), (256, 96)])
def test_products_outside_the_range(hqr_lib, cuda, nb, first, a, low, dtype):
    import paper_1110_1553_amd as h

    params = h.make_params(nb=nb, p=1, a=a, low=low)
    M, N = 2 * nb + 40, first + 12
    pairs, tol = TYPES[dtype]
    tol = tol or 10.0 * np.sqrt(M * N) * 2.0 ** -24
    G = inputs.gaussian(M, N, 91).astype(np.float32).astype(np.float64)  # exact in both types
    G[:, -1] = G[:, first]
    ref = oq.sign_normalize(oq.r_factor(G))
    for most, last in pairs:
        e = np.where(np.arange(N) < first, 0, most)
        e[-1] = last
        R = run(np.ldexp(G, e), dtype, params)
        assert np.all(np.isfinite(R)), (most, last)
        R = oq.sign_normalize(np.ldexp(R, -e))
        err = (np.linalg.norm(R - ref, axis=0) / np.linalg.norm(ref, axis=0)).max()
        print("nb %d from %d %s %s 2^%d, last 2^%d: column error %.2e" % (nb, first, low, dtype, most, last, err),
              flush=True)
        assert err <= tol, (most, last, err)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("a,low", [(65535, "flat"), (1, "binary")])
def test_identity_reflector_and_infinity(hqr_lib, cuda, a, low, dtype):
    import paper_1110_1553_amd as h

    A = inputs.gaussian(150, 2, 92)
    A[1:, 0] = 0.0
    A[0] = 2.0, 3.0
    A[5, 1] = np.inf
    print("infinity, %s %s" % (low, dtype), flush=True)
    R = run(A, dtype, h.make_params(nb=64, p=1, a=a, low=low))
    assert R[0, 0] == 2.0 and R[0, 1] == 3.0 and not np.isfinite(R[1, 1])
