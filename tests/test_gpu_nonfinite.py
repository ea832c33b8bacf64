"""NaN and infinity below the diagonal reach the pivot of their row and no
earlier one: the reported column is that row's, at the edges of the column
quads, 16-column panels, 32-column panels and tiles of the factorizations."""
import numpy as np
import pytest

import spd_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (row, column): in a quad, across quads, panels and tiles
AT = [(1, 0), (3, 1), (5, 2), (7, 4), (15, 12), (16, 0), (18, 17), (31, 16), (33, 3), (63, 62), (64, 1), (127, 20), (130, 129),
      (200, 150), (299, 3)]


@pytest.fixture(scope="module")
def tc():
    import paper_1402_6601_amd as t
    t.load()
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to the gpu-marked tests")
    return t


def _with(A, r, c, v):
    B = np.array(A)
    B[r, c] = B[c, r] = v
    return B


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("nb", [64, 128, 208])
def test_single_matrix(tc, nb, value):
    A, b = spd_inputs.spd_matrix_and_rhs(300, 11, nrhs=1)
    for r, c in AT:
        print("case nb=%d (%d, %d) %r" % (nb, r, c, value), flush=True)
        W = torch.from_numpy(_with(A, r, c, value)).cuda()
        assert tc.factor_(W.clone(), nb) == r + 1
        X = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
        assert tc.factor_solve_(W.clone(), X, nb) == r + 1


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_compact_batch(tc, value):
    n = 300
    A, b = spd_inputs.spd_matrix_and_rhs(n, 12, nrhs=1)
    As = np.stack([_with(A, r, c, value) for r, c in AT] + [A])
    count = len(As)
    W = torch.from_numpy(As.reshape(-1)).cuda()
    X = torch.from_numpy(np.tile(b[:, 0], count)).cuda()
    info = tc.factor_solve_batched_(W, np.arange(count) * n * n, [n] * count, X, np.arange(count) * n, [n] * count,
                                    [304] * count, 1)
    assert list(info) == [r + 1 for r, _ in AT] + [0]
