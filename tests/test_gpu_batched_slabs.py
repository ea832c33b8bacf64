"""The compact batched factorization at the edges of its pieces: 16-column
halves and 32-column panels, 32-row blocks of a wavefront, 128-row slabs; with
one, four (fused forward solve) and five (solved after) right-hand sides;
breakdown columns on either side of those edges."""
import numpy as np
import pytest

import oracle
import spd_inputs
from tests.test_gpu_batched import TOL, _nb_single, _run, tc  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EDGES = [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 65, 127, 128, 129, 143, 144, 145, 159, 160, 161, 255, 257, 289, 384, 416,
         500, 512]


@pytest.mark.parametrize("nrhs", [1, 4, 5])
def test_slab_edges(tc, nrhs):  # noqa: F811
    _, As, bs = spd_inputs.batched_systems(len(EDGES), 21, nrhs, sizes=EDGES)
    info, Ls, Xs = _run(tc, As, bs, [_nb_single(n) for n in EDGES])
    assert not np.any(info)
    for A, b, L, X in zip(As, bs, Ls, Xs):
        Lo = oracle.cholesky(A)
        assert oracle.factor_error(L, Lo) <= TOL
        assert oracle.backward_error(A, L) <= 10.0
        xo = np.stack([oracle.potrs(Lo, b[:, j]) for j in range(nrhs)], axis=1)
        assert np.max(np.abs(X - xo)) <= TOL * np.max(np.abs(xo))


def test_slab_breakdown(tc):  # noqa: F811
    n, cols = 300, [0, 3, 4, 15, 16, 31, 32, 127, 128, 160, 299]
    _, As, bs = spd_inputs.batched_systems(2 * len(cols) + 1, 22, 1, sizes=[n] * (2 * len(cols) + 1))
    for k, j in enumerate(cols):
        As[2 * k][j, j] = -4.0
        As[2 * k + 1][j, j] = float("nan")
    info, Ls, _ = _run(tc, As, bs, [_nb_single(n)] * len(As))
    assert list(info) == [j + 1 for j in cols for _ in range(2)] + [0]
    assert oracle.factor_error(Ls[-1], oracle.cholesky(As[-1])) <= TOL
