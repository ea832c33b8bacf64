"""Launches that factor with smaller tiles than the caller's.

A single-system factorization (alone or merged with the solve) at tiles that
are a multiple of 128 runs at tiles of 128 up to a bounded order, the merged
launch's solve at the caller's; tiles of at most 128 are factored in LDS
together with the inverse that the merged launch's TRSMs apply.  Against the
oracle at the edges of the 16-column panels, of the 32-row strips and 64 x 64
blocks of the tile kernels, and of the tiles; bitwise against the launches
that take the same path (other claim orders, the traced plan at the same
tiles, factorization and solve apart).
"""
import numpy as np
import pytest

import oracle
import spd_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10  # the FP64 target of the other parity tests


@pytest.fixture(scope="module")
def tc():
    import paper_1402_6601_amd as t
    t.load()
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to the gpu-marked tests")
    return t


def _merged(tc, A, b, nb, **kw):
    W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
    X = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
    info = tc.factor_solve_(W, X, nb, **kw)
    torch.cuda.synchronize()
    return info, np.tril(W.cpu().numpy().T), X.cpu().numpy().T


SIZES = [(15, 16), (16, 16), (31, 32), (33, 48), (65, 64), (113, 112), (127, 128), (128, 128), (129, 128), (150, 80),
         (257, 128), (385, 256), (511, 256), (640, 512), (900, 384), (1301, 512)]


@pytest.mark.parametrize("n,nb", SIZES)
def test_merged_matches_oracle(tc, n, nb):
    print("case n=%d nb=%d" % (n, nb), flush=True)
    A, b = spd_inputs.spd_matrix_and_rhs(n, n + nb, nrhs=3)
    info, L, X = _merged(tc, A, b, nb)
    assert info == 0
    Lo = oracle.cholesky(A)
    assert oracle.factor_error(L, Lo) <= TOL
    assert oracle.backward_error(A, L) <= 10.0
    xo = np.stack([oracle.potrs(Lo, b[:, j]) for j in range(3)], axis=1)
    assert np.max(np.abs(X - xo)) <= TOL * np.max(np.abs(xo))
    # the same bits under another claim order, and from the two launches
    info, L2, X2 = _merged(tc, A, b, nb, policy=tc.POLICY_RANDOM, seed=5)
    assert info == 0 and np.array_equal(L, L2) and np.array_equal(X, X2)
    W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
    assert tc.factor_(W, nb, inv_trsm=True) == 0
    Xs = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
    tc.solve_(W, Xs, nb)
    assert np.array_equal(np.tril(W.cpu().numpy().T), L) and np.array_equal(Xs.cpu().numpy().T, X)
    # substitution, merged and apart
    info, L3, X3 = _merged(tc, A, b, nb, subst=True)
    W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
    assert info == 0 and tc.factor_(W, nb) == 0
    Xs = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
    tc.solve_(W, Xs, nb, subst=True)
    assert np.array_equal(np.tril(W.cpu().numpy().T), L3) and np.array_equal(Xs.cpu().numpy().T, X3)
    assert oracle.factor_error(L3, Lo) <= TOL


@pytest.mark.parametrize("n,nb", [(300, 64), (500, 128), (400, 512)])
def test_traced_plan(tc, n, nb):
    """A traced launch runs the queried plan; at tiles of at most 128 that is the same arithmetic."""
    A, b = spd_inputs.spd_matrix_and_rhs(n, 9, nrhs=2)
    trace = torch.zeros(4 * tc.plan_query(tc.OP_FACTOR_SOLVE, n, nb)["nitem"], dtype=torch.int64, device="cuda")
    info, L, X = _merged(tc, A, b, nb, trace=trace)
    assert info == 0 and oracle.factor_error(L, oracle.cholesky(A)) <= TOL
    assert int((trace.view(-1, 4)[:, 2] > 0).sum()) == trace.numel() // 4
    if nb <= 128:
        info, L2, X2 = _merged(tc, A, b, nb)
        assert info == 0 and np.array_equal(L, L2) and np.array_equal(X, X2)


@pytest.mark.parametrize("j", [0, 3, 4, 15, 16, 63, 127, 128, 131, 255, 299])
def test_breakdown_column(tc, j):
    """The first pivot that is not positive, at the edges of column quads, panels and tiles: negative and NaN."""
    n, nb = 300, 256
    A, b = spd_inputs.spd_matrix_and_rhs(n, 2, nrhs=1)
    for bad in (-4.0, float("nan")):
        Ab = np.array(A)
        Ab[j, j] = bad
        info, _, X = _merged(tc, Ab, b, nb)
        assert info == j + 1
        assert tc.factor_(torch.from_numpy(Ab).cuda(), nb) == j + 1
