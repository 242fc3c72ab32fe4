"""The work this library is used for, as measurable cases.

A case names one call of the public Python API with its sizes and options:

  factor      h.factor: QR in place, float64 or float32 tiles
  lstsq       h.lstsq: least squares, right-hand sides carried through the factorization
  ir          h.lstsq_ir: FP32 (or BF16-product) factorization refined to FP64
  apply_qt,
  apply_q     h.apply_qt / h.apply_q with a kept factorization
  solve       h.solve: new right-hand sides against a kept factorization
  batch       h.lstsq_batched: many requests planned, bound, solved and checked in one call
  graph       BatchedLstsq.run of a few small requests replayed from a captured graph

The calls overwrite their matrices, so a pass starts by copying the pristine
ones into the buffers, as a program that keeps its data does.
"""
import math

import numpy as np
import torch

import paper_1110_1553_amd as h
from paper_1110_1553_amd import inputs

# Reduction trees by name.  "hier" is the benchmark's tall-skinny tree, "hier2" the one of its
# least-squares workload, "domains" what the serving tuner picks (TS domains under Greedy).
TREES = {
    "flat": dict(p=1, a=65535, low="flat"),
    "binary": dict(p=1, a=1, low="binary"),
    "greedy": dict(p=1, a=1, low="greedy"),
    "domains": dict(p=1, a=4, low="greedy"),
    "hier": dict(p=8, a=4, low="greedy", high="fibonacci", coupling="chain", domino=1),
    "hier2": dict(p=4, a=2, low="greedy", high="fibonacci", coupling="chain", domino=1),
}


def listed():
    return [
        # the smallest factorization of the tests and of the smoke run: latency of a call
        {"name": "factor 512x256", "op": "factor", "M": 512, "N": 256, "nb": 64, "tree": "flat", "dtype": "f64"},
        # an ordinary matrix with no size a multiple of the tile
        {"name": "factor 4001x777", "op": "factor", "M": 4001, "N": 777, "nb": 128, "tree": "greedy", "dtype": "f64"},
        # the benchmark's tall-skinny workload
        {"name": "factor 131072x2048", "op": "factor", "M": 131072, "N": 2048, "nb": 256, "tree": "hier", "dtype": "f64"},
        # the benchmark's square workload, the largest call
        {"name": "factor 16384x16384", "op": "factor", "M": 16384, "N": 16384, "nb": 256, "tree": "flat", "dtype": "f64"},
        # single precision, square
        {"name": "factor 8192x8192 f32", "op": "factor", "M": 8192, "N": 8192, "nb": 256, "tree": "flat", "dtype": "f32"},
        # the benchmark's least-squares workload
        {"name": "lstsq 32768x2048", "op": "lstsq", "M": 32768, "N": 2048, "nb": 256, "tree": "hier2", "nrhs": 1},
        # one small request on its own
        {"name": "lstsq 1000x37", "op": "lstsq", "M": 1000, "N": 37, "nb": 64, "tree": "greedy", "nrhs": 1},
        # mixed precision with refinement
        {"name": "ir 16384x1024", "op": "ir", "M": 16384, "N": 1024, "nb": 256, "tree": "hier", "precision": "fp32"},
        # projections of a block of vectors, an odd number of them
        {"name": "apply_qt 32768x1024 x200", "op": "apply_qt", "M": 32768, "N": 1024, "nb": 256, "tree": "domains",
         "nrhs": 200},
        # the thin Q itself: Q times the first columns of the identity
        {"name": "apply_q 16384x512 x512", "op": "apply_q", "M": 16384, "N": 512, "nb": 256, "tree": "domains", "nrhs": 512},
        # a later right-hand side for a factorization that the server kept
        {"name": "solve 16384x512", "op": "solve", "M": 16384, "N": 512, "nb": 256, "tree": "domains", "nrhs": 1},
        # a batch of the serving workload's requests (rows up to 16384, columns up to 512), the whole call
        {"name": "batch 48", "op": "batch", "count": 48, "shapes": 5, "nb": 256, "tree": "domains"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["factor", "factor", "factor", "factor32", "lstsq", "lstsq", "ir", "apply_qt", "apply_q", "solve",
                     "batch", "graph"])
    if op == "batch":
        return {"op": "batch", "count": rng.randint(4, 60), "shapes": rng.randint(10, 10 ** 6), "nb": 256,
                "tree": rng.choice(["domains", "greedy"])}
    if op == "graph":
        return {"op": "graph", "count": rng.randint(2, 12), "shapes": rng.randint(10, 10 ** 6), "nb": 64, "tree": "greedy"}
    nb = rng.choice([64, 128, 256, 256])
    tall = rng.random() < 0.7
    if op == "factor":
        N = _log(rng, 16, 4096)
        M = N + (_log(rng, 16, 131072 if N <= 1024 else 32768) if tall else rng.randint(0, N))
        # a flat tree is a serial chain of tile rows: for matrices that are not much taller than wide
        tree = rng.choice(["flat", "greedy"] if M < 4 * N else ["hier", "hier2", "domains", "greedy", "binary"])
        return {"op": "factor", "M": M, "N": N, "nb": 256 if M > 16384 else nb, "tree": tree, "dtype": "f64"}
    if op == "factor32":
        N = _log(rng, 16, 2048)
        M = N + (_log(rng, 16, 8192) if tall else rng.randint(0, N))
        return {"op": "factor", "M": M, "N": N, "nb": nb, "tree": rng.choice(["flat", "domains"]), "dtype": "f32"}
    if op == "ir":
        N = _log(rng, 32, 2048)
        M = N + _log(rng, 256, 32768)
        return {"op": "ir", "M": M, "N": N, "nb": 256 if M > 16384 else nb, "tree": rng.choice(["hier", "domains"]),
                "precision": rng.choice(["fp32", "fp32", "bf16"])}
    N = _log(rng, 16, 2048)
    M = N + _log(rng, 16, 65536)
    nrhs = 1 if rng.random() < 0.5 else _log(rng, 1, 400)
    return {"op": op, "M": M, "N": N, "nb": 256 if M > 16384 else nb,
            "tree": rng.choice(["hier2", "domains", "greedy"]), "nrhs": nrhs}


def _params(case):
    return h.make_params(nb=case["nb"], precision=case.get("precision", "fp64"), **TREES[case["tree"]])


def _shapes(case):
    """(rows, columns) of a batch's requests."""
    if case["op"] == "graph":
        m, n = inputs.request_shapes(case["count"], case["shapes"], 64, 2048, 8, 128)
    else:
        m, n = inputs.request_shapes(case["count"], case["shapes"])
    return [(int(a), int(b)) for a, b in zip(m, n)]


def _randn(shape, seed, dtype=torch.float64):
    """iid N(0,1), column-major."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(tuple(reversed(shape)), generator=g, device="cuda", dtype=dtype).t()


def _matrices(case, seed):
    """Pristine A and B of a single-problem case."""
    M, N = case["M"], case["N"]
    dtype = torch.float32 if case.get("dtype") == "f32" else torch.float64
    A = _randn((M, N), 2 * seed + 1, dtype)
    op, r = case["op"], case.get("nrhs", 1)
    if op == "factor":
        return A, None
    if op in ("lstsq", "ir", "solve"):
        # a regression: columns of different scale, a right-hand side that the columns explain up to noise
        A = A * torch.logspace(0.0, -2.0, N, device="cuda", dtype=dtype)
        B = (A @ _randn((N, r), 2 * seed + 2)).t().contiguous().t()
        return A, B + 0.1 * _randn((M, r), 2 * seed + 3)
    if op == "apply_q" and r <= N:
        return A, torch.eye(r, M, device="cuda", dtype=dtype).t()
    return A, _randn((M, r), 2 * seed + 2)


def _requests(case, seed):
    """One flat buffer with every request's A and another with every b, and the views of them."""
    shapes = _shapes(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    A = torch.randn(sum(m * n for m, n in shapes), generator=g, device="cuda", dtype=torch.float64)
    B = torch.randn(sum(m for m, _ in shapes), generator=g, device="cuda", dtype=torch.float64)
    return shapes, A, B


def _views(shapes, A, B):
    As, Bs, a, b = [], [], 0, 0
    for m, n in shapes:
        As.append(A[a:a + m * n].view(n, m).t())
        Bs.append(B[b:b + m].view(1, m).t())
        a, b = a + m * n, b + m
    return As, Bs


def prepare(case, seed):
    op, params = case["op"], _params(case)
    s = {"op": op, "params": params}
    if op in ("batch", "graph"):
        shapes, s["A0"], s["B0"] = _requests(case, seed)
        s["A"], s["B"] = s["A0"].clone(), s["B0"].clone()
        s["As"], s["Bs"] = _views(shapes, s["A"], s["B"])
        s["x"] = [b[:n] for b, (_, n) in zip(s["Bs"], shapes)]
        if op == "graph":
            stream = torch.cuda.Stream()
            stream.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(stream):
                s["solver"] = h.BatchedLstsq(s["As"], s["Bs"], params)
                s["solver"].run()
            torch.cuda.current_stream().wait_stream(stream)
            torch.cuda.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                s["solver"].run()
        return s
    M, N, r = case["M"], case["N"], case.get("nrhs", 1)
    s["M"], s["N"] = M, N
    s["A0"], s["B0"] = _matrices(case, seed)
    if op == "ir":
        s["b"] = s["B0"].reshape(-1).contiguous()
        return s
    f32 = case.get("dtype") == "f32"
    s["A"] = s["A0"].clone()
    s["work"] = h.Workspace(M, N, params, nrhs=r if op == "lstsq" else 0, f32=f32)
    if op != "factor":
        s["B"] = s["B0"].clone()
    if op in ("apply_qt", "apply_q", "solve"):
        h.factor(s["A"], params, work=s["work"])
        s["bwork"] = h.ApplyWorkspace(M, r, params)
        s["A0"] = None
    return s


def run(s):
    op, params = s["op"], s["params"]
    if op == "factor":
        s["A"].copy_(s["A0"])
        h.factor(s["A"], params, work=s["work"], check=False)
        return {"A": s["A"]}
    if op == "lstsq":
        s["A"].copy_(s["A0"])
        s["B"].copy_(s["B0"])
        h.lstsq(s["A"], s["B"], params, work=s["work"], check=False)
        return {"x": s["B"][:s["N"]], "residual": s["B"][s["N"]:], "A": s["A"]}
    if op == "ir":
        x, r, _ = h.lstsq_ir(s["A0"], s["b"], params, residual=True)
        return {"x": x, "r": r}
    if op in ("apply_qt", "apply_q"):
        s["B"].copy_(s["B0"])
        (h.apply_qt if op == "apply_qt" else h.apply_q)(s["B"], s["M"], s["N"], params, s["work"], bwork=s["bwork"],
                                                        check=False)
        return {"B": s["B"]}
    if op == "solve":
        s["B"].copy_(s["B0"])
        h.solve(s["B"], s["M"], s["N"], params, s["work"], bwork=s["bwork"], check=False)
        return {"x": s["B"][:s["N"]], "residual": s["B"][s["N"]:]}
    s["A"].copy_(s["A0"])
    s["B"].copy_(s["B0"])
    if op == "batch":
        h.lstsq_batched(s["As"], s["Bs"], params)
    else:
        s["graph"].replay()
    return {"x": s["x"], "A": s["A"], "B": s["B"]}


def _qr_flops(m, n):
    return 2.0 * m * n * n - 2.0 * n ** 3 / 3.0


def work(case):
    """Householder counts; every input read once and every output written once."""
    op = case["op"]
    if op in ("batch", "graph"):
        shapes = _shapes(case)
        return {"bytes": 16.0 * sum(m * n + m for m, n in shapes),
                "flops": float(sum(_qr_flops(m, n) + 4.0 * m * n - n * n for m, n in shapes))}
    M, N, r = case["M"], case["N"], case.get("nrhs", 1)
    if op == "factor":
        return {"bytes": 2.0 * M * N * (4 if case["dtype"] == "f32" else 8), "flops": _qr_flops(M, N)}
    apply = 4.0 * M * N * r - 2.0 * N * N * r
    if op == "lstsq":
        return {"bytes": 16.0 * (M * N + M * r), "flops": _qr_flops(M, N) + apply + N * N * r}
    if op == "ir":
        # the factorization and one residual of the original matrix
        return {"bytes": 8.0 * (M * N + 2 * M + N), "flops": _qr_flops(M, N) + apply + N * N + 4.0 * M * N}
    return {"bytes": 8.0 * (M * N + 2 * M * r), "flops": apply + (N * N * r if op == "solve" else 0)}


def _tiled(A, nb, tree, B, trans):
    """The tiled factorization of A (M x N) with a flat or binary tree, tile by tile with LAPACK's
    Householder QR in 64 bits, and Q^T B (trans) or Q B.  Returns the factored A and that."""
    M, N = A.shape
    mt, nt = -(-M // nb), -(-N // nb)
    P = torch.zeros((mt * nb, nt * nb), dtype=torch.float64)
    P[:M, :N] = A
    ops = []  # (first rows, second rows or None, reflectors, tau)

    def rows(i):
        return slice(i * nb, (i + 1) * nb)

    def apply(X, op, transpose):
        i, j, V, tau = op
        if X.shape[1] == 0:
            return
        if j is None:
            X[rows(i)] = torch.ormqr(V, tau, X[rows(i)].contiguous(), True, transpose)
            return
        C = torch.ormqr(V, tau, torch.cat([X[rows(i)], X[rows(j)]]), True, transpose)
        X[rows(i)], X[rows(j)] = C[:nb], C[nb:]

    for k in range(nt):
        c = slice(k * nb, (k + 1) * nb)
        right = P[:, (k + 1) * nb:]

        def triangle(i):
            V, tau = torch.geqrf(P[rows(i), c].contiguous())
            P[rows(i), c] = V
            ops.append((i, None, V, tau))
            apply(right, ops[-1], True)

        def kill(i, j, square):
            """Row i's triangle on top of row j's square or triangle."""
            V, tau = torch.geqrf(torch.cat([P[rows(i), c].triu(), P[rows(j), c] if square else P[rows(j), c].triu()]))
            P[rows(i), c] = V[:nb].triu() + P[rows(i), c].tril(-1)
            P[rows(j), c] = V[nb:] if square else V[nb:].triu() + P[rows(j), c].tril(-1)
            ops.append((i, j, V, tau))
            apply(right, ops[-1], True)

        if tree == "flat":
            triangle(k)
            for j in range(k + 1, mt):
                kill(k, j, True)
        else:
            for i in range(k, mt):
                triangle(i)
            step = 1
            while step < mt - k:
                for i in range(k, mt - step, 2 * step):
                    kill(i, i + step, False)
                step *= 2
    X = None
    if B is not None:
        X = torch.zeros((mt * nb, B.shape[1]), dtype=torch.float64)
        X[:M] = B
        for op in (ops if trans else reversed(ops)):
            apply(X, op, trans)
        X = X[:M]
    return P[:M, :N], X


def _ls(A, B):
    return torch.linalg.lstsq(A, B, driver="gels").solution


def exact(case, seed):
    """What `run` returns, in 64 bits with LAPACK.  The reflectors, the signs of R and the last rows of Q^T B
    depend on the elimination order, which is spelled out above for the flat and the binary tree; least-squares
    solutions do not depend on it."""
    op = case["op"]
    if op in ("batch", "graph"):
        shapes, A, B = _requests(case, seed)
        if sum(_qr_flops(m, n) for m, n in shapes) > 1.5e11:
            return None
        As, Bs = _views(shapes, A.cpu(), B.cpu())
        return {"x": [_ls(a, b) for a, b in zip(As, Bs)], "A": None, "B": None}
    M, N = case["M"], case["N"]
    if op == "factor" and (case["tree"] not in ("flat", "binary") or _qr_flops(M, N) > 8e11):
        return None
    if _qr_flops(M, N) > 1e12:
        return None
    A, B = _matrices(case, seed)
    A, B = A.cpu().double(), None if B is None else B.cpu().double()
    if op == "factor":
        return {"A": _tiled(A, case["nb"], case["tree"], None, True)[0]}
    if op in ("apply_qt", "apply_q"):
        if case["tree"] not in ("flat", "binary"):
            return None
        return {"B": _tiled(A, case["nb"], case["tree"], B, op == "apply_qt")[1]}
    x = _ls(A, B)
    if op == "ir":
        return {"x": x.reshape(-1), "r": (B - A @ x).reshape(-1)}
    return {"x": x, "residual": None, "A": None} if op == "lstsq" else {"x": x, "residual": None}
