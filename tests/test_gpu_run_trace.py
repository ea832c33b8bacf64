"""A trace of the plan that ordinary launches run: every work item of the
queried run plan recorded, bitwise the untraced launch's results."""
import numpy as np
import pytest

import spd_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(300, 64), (700, 256), (1301, 512), (1000, 192)])
@pytest.mark.parametrize("merged", [True, False])
def test_trace_of_the_run_plan(n, nb, merged):
    import paper_1402_6601_amd as tc
    tc.load()
    assert torch.cuda.is_available()
    A, b = spd_inputs.spd_matrix_and_rhs(n, n, nrhs=2)
    pol = tc.POLICY_LIST | tc.PLAN_RUN
    plan = tc.plan_query(tc.OP_FACTOR_SOLVE if merged else tc.OP_FACTOR, n, nb, pol)

    def run(**kw):
        W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
        X = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
        info = tc.factor_solve_(W, X, nb, **kw) if merged else tc.factor_(W, nb, **kw)
        assert info == 0
        return W.cpu().numpy(), X.cpu().numpy()

    trace = torch.zeros(4 * plan["nitem"], dtype=torch.int64, device="cuda")
    W1, X1 = run(policy=pol, trace=trace)
    W2, X2 = run()
    W3, X3 = run(policy=pol)
    assert np.array_equal(W1, W2) and np.array_equal(X1, X2)
    assert np.array_equal(W1, W3) and np.array_equal(X1, X3)
    tr = trace.cpu().numpy().reshape(-1, 4)
    assert np.all(tr[:, 2] >= tr[:, 1]) and np.all(tr[:, 0] > 0)
    seen = np.bincount((tr[:, 3] & 0xffffffff).astype(np.int64), minlength=plan["ntask"])
    assert np.array_equal(seen, plan["parts"][:plan["ntask"]])
    # one item's room less is refused
    with pytest.raises(tc.TcholError):
        run(policy=pol, trace=trace[:-4].clone())
