"""BF16-update factorization at the edges of its diagonal blocks (16, 128 and
the shared tiles above): the first solution, before any refinement, is as
accurate as with FP32 updates, and the refinement takes at most one step more."""
import numpy as np
import pytest

import oracle
import spd_inputs
from tests.test_gpu_mixed import TARGET, _mixed, tc  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(500, 112), (777, 128), (900, 144), (1100, 256), (1300, 272), (1500, 384), (1700, 496)])
def test_first_solution_and_refinement(tc, n, nb):  # noqa: F811
    print("case n=%d nb=%d" % (n, nb), flush=True)
    A, b = spd_inputs.spd_matrix_and_rhs(n, nb, nrhs=4, shift=1e-4)
    _, _, _, X32 = _mixed(tc, A, b, nb, lowp=1, maxit=0)
    _, _, _, X16 = _mixed(tc, A, b, nb, lowp=2, maxit=0)
    e32, e16 = (oracle.solve_backward_error(A, X, b).max() for X in (X32, X16))
    assert e16 <= 4.0 * e32, (e16, e32)  # the bound of the check at order 2048
    _, it32, _, _ = _mixed(tc, A, b, nb, lowp=1)
    rc, it16, _, X = _mixed(tc, A, b, nb, lowp=2)
    assert rc == 0 and it16 <= it32 + 1, (it32, it16)
    assert np.all(oracle.solve_backward_error(A, X, b) <= TARGET)
