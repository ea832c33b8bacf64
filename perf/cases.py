"""The work that a program has this library do, as timed cases.

Every case is one call (or one forward and backward) through the package's
public entry points on symmetric positive definite systems of the family the
benchmark and the tests use, A = B B^T / n + shift I with B uniform in
[-1, 1], over the orders, tile sizes, right-hand sides, batch shapes and
precisions that they use.

The entry points work in place, so a pass first copies the pristine matrix
and right-hand sides into the buffers it hands over, as a program does that
factors a new matrix on every step.  The workspace is kept across passes.
"""
import math

import numpy as np
import torch

import paper_1402_6601_amd as tc
from paper_1402_6601_amd import autotune

#: Largest order whose factorization in 64 bits on the host stays well under twenty seconds.
EXACT_ORDER = 16384


def listed():
    return [
        # a single small system solved at once: latency, launches and host work are all there is
        {"name": "factor_solve_300", "path": "factor_solve", "n": 300, "nb": 64, "nrhs": 3},
        # the small benchmark system (one right-hand side)
        {"name": "factor_solve_1024", "path": "factor_solve", "n": 1024, "nb": 128, "nrhs": 1},
        # the paper's smaller matrix, at its tile size
        {"name": "factor_solve_8192", "path": "factor_solve", "n": 8192, "nb": 512, "nrhs": 16},
        # the headline system of the benchmark
        {"name": "factor_solve_32768", "path": "factor_solve", "n": 32768, "nb": 512, "nrhs": 16},
        # new right-hand sides against a factor kept from before (the paper's larger matrix)
        {"name": "solve_16384", "path": "solve", "n": 16384, "nb": 512, "nrhs": 16},
        # the batched benchmark: thousands of systems of mixed orders, in both storage types
        {"name": "batched_4096", "path": "batched", "count": 4096, "lo": 16, "hi": 512, "nrhs": 4, "fp32": False,
         "sizes": 4},
        {"name": "batched_f32_4096", "path": "batched", "count": 4096, "lo": 16, "hi": 512, "nrhs": 4, "fp32": True,
         "sizes": 4},
        # a batch of a few hundred small systems, as in a local solver's inner loop
        {"name": "batched_small_512", "path": "batched", "count": 512, "lo": 16, "hi": 128, "nrhs": 1, "fp32": False,
         "sizes": 5},
        # the mixed-precision benchmark (BF16 updates, refined to a backward error of 1e-12)
        {"name": "mixed_bf16_32768", "path": "mixed", "n": 32768, "nb": 512, "nrhs": 16, "lowp": tc.LOWP_BF16,
         "shift": 1e-4},
        # a mid-sized mixed-precision solve with FP32 updates and a ragged last tile
        {"name": "mixed_fp32_6000", "path": "mixed", "n": 6000, "nb": 384, "nrhs": 5, "lowp": tc.LOWP_FP32,
         "shift": 1e-2},
        # the adjoint of the factorization alone (the benchmark's)
        {"name": "adjoint_8192", "path": "adjoint", "n": 8192, "nb": 256},
        # forward and backward through autograd on an odd order (no 16-byte rows, ragged tiles)
        {"name": "autograd_3001", "path": "autograd", "n": 3001, "nb": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _order_and_tile(rng, lo, hi):
    """An order, any residue, and a tile size that cuts it into 3 to 64 tiles a side."""
    n = _log_int(rng, lo, hi)
    fit = [nb for nb in (64, 128, 256, 384, 512) if 3 <= -(-n // nb) <= 64]
    return n, rng.choice(fit)


def draw(rng):
    path = rng.choice(["factor_solve", "factor_solve", "solve", "batched", "batched", "mixed", "adjoint", "autograd"])
    if path == "batched":
        return {"path": path, "count": _log_int(rng, 64, 4096), "lo": 16, "hi": _log_int(rng, 64, 512),
                "nrhs": rng.choice([1, 2, 4, 4, 7]), "fp32": rng.random() < 0.4, "sizes": rng.randrange(1 << 30)}
    hi = {"factor_solve": 24000, "solve": 20000, "mixed": 20000, "adjoint": 8192, "autograd": 6000}[path]
    n, nb = _order_and_tile(rng, 300, hi)
    if path in ("adjoint", "autograd"):
        return {"path": path, "n": n, "nb": nb}
    case = {"path": path, "n": n, "nb": nb, "nrhs": _log_int(rng, 1, 16)}
    if path == "mixed":
        case["lowp"] = rng.choice([tc.LOWP_BF16, tc.LOWP_FP32])
        case["shift"] = rng.choice([1e-4, 1e-2])
    return case


# ---------------------------------------------------------------- inputs


def _uniform(gen, *shape):
    return torch.rand(*shape, generator=gen, dtype=torch.float64, device="cuda").mul_(2.0).sub_(1.0)


def _spd(gen, n, shift):
    B = _uniform(gen, n, n).mul_(n ** -0.5)
    A = torch.mm(B, B.t().contiguous())
    del B
    for r in range(0, n, 4096):  # exactly symmetric: the upper part from the lower
        s = min(n, r + 4096)
        A[r:s, s:] = A[s:, r:s].t()
        D = A[r:s, r:s]
        D.copy_(torch.tril(D) + torch.tril(D, -1).t())
    A.diagonal().add_(shift)
    return A


def _orders(case):
    return np.random.default_rng(case["sizes"]).integers(case["lo"], case["hi"] + 1, size=case["count"])


def _pack(ns, nrhs, fp32):
    """Leading dimensions and offsets as the batched entry points' fast paths take them."""
    lda = (ns + 6) // 4 * 4 if fp32 else (ns + 1) // 2 * 2
    a_off = np.concatenate([[0], np.cumsum(lda * ns)])
    b_off = np.concatenate([[0], np.cumsum(ns * nrhs)])
    return lda, a_off[:-1], b_off[:-1], int(a_off[-1]), int(b_off[-1])


def _batch(gen, case):
    ns = _orders(case)
    lda, a_off, b_off, na, nbt = _pack(ns, case["nrhs"], case["fp32"])
    dt = torch.float32 if case["fp32"] else torch.float64
    A = torch.zeros(na, dtype=dt, device="cuda")
    raw = _uniform(gen, int((ns * ns).sum()))
    at = 0
    for n, o, l in zip(ns.tolist(), a_off.tolist(), lda.tolist()):
        B = raw[at:at + n * n].view(n, n)
        at += n * n
        S = torch.mm(B, B.t().contiguous()).mul_(1.0 / n)
        S.diagonal().add_(1.0)
        A[o:o + n * l].view(n, l)[:, :n].copy_(S)
    return ns, lda, a_off, b_off, A, _uniform(gen, nbt).to(dt)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    path = case["path"]
    if path == "batched":
        return _batch(gen, case)
    n = case["n"]
    A = _spd(gen, n, case.get("shift", 1.0))
    if path in ("adjoint", "autograd"):
        return A, torch.randn(n, n, generator=gen, dtype=torch.float64, device="cuda").tril_()
    return A, _uniform(gen, case["nrhs"], n)


def prepare(case, seed):
    path = case["path"]
    if path == "batched":
        ns, lda, a_off, b_off, A, B = _inputs(case, seed)
        nb = autotune.tile_sizes(ns)
        need = (tc.batched_f32_workspace_bytes(ns, nb, case["nrhs"]) if case["fp32"]
                else tc.batched_workspace_bytes(ns, nb))
        return {"case": case, "A": A, "B": B, "W": torch.empty_like(A), "X": torch.empty_like(B), "ns": ns, "nb": nb,
                "lda": lda, "a_off": a_off, "b_off": b_off, "ws": _workspace(need)}
    n, nb = case["n"], case["nb"]
    A, B = _inputs(case, seed)
    s = {"case": case, "A": A, "B": B}
    if path == "factor_solve":
        s.update(W=torch.empty_like(A), X=torch.empty_like(B),
                 ws=_workspace(tc.factor_solve_workspace_bytes(n, nb, case["nrhs"])))
    elif path == "mixed":
        s.update(X=torch.empty_like(B), ws=_workspace(tc.mixed_workspace_bytes(n, nb, case["nrhs"], case["lowp"])))
    elif path == "solve":  # the factor is what the program kept; right-hand sides come as the columns of (n, nrhs)
        if tc.factor_(A, nb) != 0:
            raise RuntimeError("the matrix did not factor")
        s.update(B=B.t().contiguous(), ws=_workspace(tc.workspace_bytes(tc.OP_SOLVE, n, nb, case["nrhs"])))
    elif path == "adjoint":
        if tc.factor_(A, nb) != 0:
            raise RuntimeError("the matrix did not factor")
        s.update(B=B.t().contiguous(), W=torch.empty_like(B), ws=_workspace(tc.workspace_bytes(tc.OP_BACKWARD, n, nb)))
    else:
        A.requires_grad_(True)
    return s


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda")


# ---------------------------------------------------------------- one pass


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "factor_solve":
        s["W"].copy_(s["A"])
        s["X"].copy_(s["B"])
        info = tc.factor_solve_(s["W"], s["X"], case["nb"], ws=s["ws"])
        return [s["W"], s["X"], info]
    if path == "solve":
        return [tc.solve(s["A"], s["B"], case["nb"], ws=s["ws"])]
    if path == "batched":
        s["W"].copy_(s["A"])
        s["X"].copy_(s["B"])
        call = tc.factor_solve_batched_f32_ if case["fp32"] else tc.factor_solve_batched_
        info = call(s["W"], s["a_off"], s["lda"], s["X"], s["b_off"], s["ns"], s["nb"], case["nrhs"], ws=s["ws"])
        return [s["W"], s["X"], info]
    if path == "mixed":
        # the backward errors reported beside the solution only say that the iteration stopped below its tolerance
        s["X"].copy_(s["B"])
        rc, iters, _ = tc.solve_mixed_(s["A"], s["X"], case["nb"], lowp=case["lowp"], ws=s["ws"])
        return [s["X"], rc, iters]
    if path == "adjoint":
        s["W"].copy_(s["B"])
        rc = tc.backward_(s["A"], s["W"], case["nb"], ws=s["ws"])
        return [s["W"], rc]
    L = tc.cholesky(s["A"], case["nb"])
    (g,) = torch.autograd.grad(L, s["A"], s["B"])
    return [L.detach(), g]


# ---------------------------------------------------------------- what a pass cannot do without


def work(case):
    path = case["path"]
    if path == "batched":
        ns, size = _orders(case).astype(np.float64), 4 if case["fp32"] else 8
        k = case["nrhs"]
        # the lower triangle read and L written; the right-hand sides read and the solutions written
        return {"bytes": size * float((ns * (ns + 1) + 2 * ns * k).sum()),
                "flops": float((ns ** 3 / 3 + 2 * ns ** 2 * k).sum())}
    n, k = float(case["n"]), float(case.get("nrhs", 0))
    tri = 8 * n * (n + 1) / 2
    if path == "factor_solve":
        return {"bytes": 2 * tri + 16 * n * k, "flops": n ** 3 / 3 + 2 * n * n * k}
    if path == "mixed":
        return {"bytes": tri + 16 * n * k, "flops": n ** 3 / 3 + 2 * n * n * k}
    if path == "solve":
        return {"bytes": tri + 16 * n * k, "flops": 2 * n * n * k}
    if path == "adjoint":
        return {"bytes": 3 * tri, "flops": 2 * n ** 3 / 3}
    return {"bytes": 3 * tri + 8 * n * n, "flops": n ** 3}


# ---------------------------------------------------------------- the same in 64 bits, by torch on the host


def _sym(M):
    return torch.tril(M) + torch.tril(M, -1).t()


def _chol_solve(L, B):
    Y = torch.linalg.solve_triangular(L, B, upper=False)
    return torch.linalg.solve_triangular(L.t(), Y, upper=True)


def _adjoint(L, G):
    """The symmetric gradient of <G, chol(A)> with respect to A (G lower)."""
    P = torch.tril(L.t() @ G)
    P.diagonal().mul_(0.5)
    S = torch.linalg.solve_triangular(L.t(), P, upper=True)                     # L^-T P
    S = torch.linalg.solve_triangular(L.t(), S.t().contiguous(), upper=True).t()  # ... L^-1
    return (S + S.t()) * 0.5


def exact(case, seed):
    if case.get("n", 0) > EXACT_ORDER:
        return None
    path = case["path"]
    if path == "batched":
        ns, lda, a_off, b_off, A, B = _inputs(case, seed)
        A, B, k = A.cpu().double(), B.cpu().double(), case["nrhs"]
        for n, o, l, ob in zip(ns.tolist(), a_off.tolist(), lda.tolist(), b_off.tolist()):
            V = A[o:o + n * l].view(n, l)[:, :n]
            L = torch.linalg.cholesky(_sym(V.t()))
            V.copy_(torch.tril(V, -1) + L.t())
            R = B[ob:ob + n * k].view(k, n)
            R.copy_(torch.cholesky_solve(R.t(), L).t())
        return [A, B, np.zeros(len(ns), dtype=np.int32)]
    A, B = (t.cpu() for t in _inputs(case, seed))
    L = torch.linalg.cholesky(A)
    if path == "factor_solve":
        return [torch.tril(A, -1) + L.t(), _chol_solve(L, B.t()).t().contiguous(), 0]
    if path == "solve":
        return [_chol_solve(L, B.t())]
    if path == "mixed":
        return [_chol_solve(L, B.t()).t().contiguous(), 0, None]
    if path == "adjoint":
        G = _adjoint(L, B)
        # the column-major lower triangle is replaced; the other triangle of the buffer stays zero
        return [torch.triu(G), 0]
    return [L, _adjoint(L, B)]
