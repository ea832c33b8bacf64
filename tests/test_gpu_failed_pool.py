"""A failing system stops its own remaining work, also inside a diagonal tile
that several workgroups share: nothing after the sub-block whose pivot failed
is written, in the tile or in later ones, whatever the claim order."""
import numpy as np
import pytest

import spd_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1402_6601_amd as t
    t.load()
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to the gpu-marked tests")
    return t


@pytest.mark.parametrize("n,nb", [(500, 192), (700, 208), (1000, 448), (600, 320)])
@pytest.mark.parametrize("call", ["inverses", "substitution", "random order", "batch of one", "batch of three"])
def test_nothing_after_the_failed_sub_block(tc, n, nb, call):
    print("case n=%d nb=%d %s" % (n, nb, call), flush=True)
    A, b = spd_inputs.spd_matrix_and_rhs(n, nb, nrhs=2)
    A = np.array(A)
    j = 10
    A[j, j] = -4.0
    W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
    X = torch.from_numpy(np.ascontiguousarray(b.T)).cuda()
    if call.startswith("batch"):
        # (no 16-byte slack is needed: the orders are even)
        count = 3 if call == "batch of three" else 1
        W = W.reshape(-1).repeat(count)
        X = X.reshape(-1).repeat(count)
        info = tc.factor_solve_batched_(W, [s * n * n for s in range(count)], [n] * count, X,
                                        [s * 2 * n for s in range(count)], [n] * count, [nb] * count, 2)
        assert list(info) == [j + 1] * count
        got = W.cpu().numpy().reshape(count, n, n)
    else:
        kw = {"inverses": {}, "substitution": {"subst": True},
              "random order": {"policy": tc.POLICY_RANDOM, "seed": 4}}[call]
        assert tc.factor_solve_(W, X, nb, **kw) == j + 1
        got = W.cpu().numpy()[None]
    # the first sub-block (128 rows and columns) holds what was done before the
    # pivot failed; the rest of the matrix is as it was
    for g in got:
        untouched = np.array(A)
        untouched[:128, :128] = g[:128, :128]
        assert np.array_equal(g, untouched)
