"""Diagonal tiles above 128, whose POTRF several workgroups share.

Their updates run in 64 x 64 blocks: tiles at the edges of the sub-blocks (128)
and of those blocks, which no 128 divides (others may be factored at smaller
tiles), against the oracle.  And the BF16-update factorization at an order
above the one from which it factors its diagonal blocks column by column, with
a ragged last tile: the solution's backward error.
"""
import numpy as np
import pytest

import oracle
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


@pytest.mark.parametrize("nb", [144, 192, 208, 272, 336, 448, 464, 496])
def test_shared_potrf_matches_oracle(tc, nb):
    n = 2 * nb + 137
    print("case n=%d nb=%d" % (n, nb), flush=True)
    A, _ = spd_inputs.spd_matrix_and_rhs(n, nb, nrhs=1)
    W = torch.from_numpy(np.ascontiguousarray(A)).cuda()
    assert tc.factor_(W, nb) == 0
    L = np.tril(W.cpu().numpy().T)
    assert oracle.factor_error(L, oracle.cholesky(A)) <= 1e-10  # the FP64 target of the other parity tests
    assert oracle.backward_error(A, L) <= 10.0


def test_bf16_updates_at_a_large_order(tc):
    n, nb, nrhs = 24640, 512, 3
    gen = torch.Generator(device="cuda").manual_seed(9)
    G = torch.rand(n, n, generator=gen, dtype=torch.float64, device="cuda").mul_(2.0).sub_(1.0)
    A = torch.mm(G, G.t().contiguous()).div_(n)
    A.diagonal().add_(1e-2)
    A = torch.tril(A) + torch.tril(A, -1).t()
    A = A.contiguous()
    B = torch.rand(nrhs, n, generator=gen, dtype=torch.float64, device="cuda").mul_(2.0).sub_(1.0)
    X = B.clone()
    print("case n=%d nb=%d" % (n, nb), flush=True)
    rc, iters, berr = tc.solve_mixed_(A, X, nb, lowp=tc.LOWP_BF16)
    assert rc == 0 and iters >= 1 and float(np.max(berr)) <= 1e-12
    R = B.t() - torch.mm(A, X.t().contiguous())
    norm_a = float(A.abs().sum(dim=1).max())
    eta = R.abs().amax(dim=0) / (norm_a * X.abs().amax(dim=1) + B.abs().amax(dim=1))
    # the rounding of a residual of n products, in the library's and here
    assert float(eta.max()) <= 1e-12 + 2 * (n + 1) * 2.0 ** -53
