"""A workspace that holds the queried plan and no more: the launch runs that
plan (bitwise the traced launch, which always does), one byte block less is
refused, and the size the query gives runs the other one.  Through the C ABI:
the Python wrappers replace a workspace that is smaller than the query's."""
import ctypes

import numpy as np
import pytest

import oracle
import spd_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(700, 256), (1301, 512), (2000, 384)])
def test_queried_plan_in_its_own_workspace(n, nb):
    import paper_1402_6601_amd as tc
    lib = tc.load()
    assert torch.cuda.is_available()
    A, b = spd_inputs.spd_matrix_and_rhs(n, n, nrhs=2)
    queried = tc.batched_workspace_bytes([n], [nb])  # the substituting launch's plan
    full = tc.factor_solve_workspace_bytes(n, nb, 2)
    assert full > queried
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    o = tc.Opts()
    o.subst = 1

    def run(nbytes):
        W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
        X = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
        rc = lib.tchol_factor_solve(ctypes.c_void_p(W.data_ptr()), n, nb, ctypes.c_void_p(X.data_ptr()), 2,
                                    ctypes.c_void_p(ws.data_ptr()), nbytes, None, ctypes.byref(o))
        torch.cuda.synchronize()
        return rc, np.tril(W.cpu().numpy().T), X.cpu().numpy().T

    assert run(queried - 256)[0] == -7
    trace = torch.zeros(4 * tc.batched_plan_query([n], [nb])["nitem"], dtype=torch.int64, device="cuda")
    W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
    X = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
    assert tc.factor_solve_(W, X, nb, subst=True, trace=trace) == 0
    rc, L, Y = run(queried)
    assert rc == 0 and np.array_equal(L, np.tril(W.cpu().numpy().T)) and np.array_equal(Y, X.cpu().numpy().T)
    Lo = oracle.cholesky(A)
    xo = np.stack([oracle.potrs(Lo, b[:, j]) for j in range(2)], axis=1)
    for rc, L, Y in (run(queried), run(full)):
        assert rc == 0 and oracle.factor_error(L, Lo) <= 1e-10
        assert np.max(np.abs(Y - xo)) <= 1e-10 * np.max(np.abs(xo))
