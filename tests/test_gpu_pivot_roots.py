"""The square roots of the pivots: L_cc = sqrt(d) to the last bit.

A diagonal matrix factors into the square roots of its entries, so L_cc shows
the arithmetic of the pivot alone: a reciprocal square root to an ulp, times d,
with one correction of the residual d - l^2.  The corrected value is within
2^-52 of half an ulp of sqrt(d), so it is the rounded square root unless sqrt(d)
lies that close to the middle of two numbers, which none of these entries does
(checked below).  Without the correction about one in five is an ulp off.
Entries from the smallest subnormal numbers up.
"""
import decimal

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1402_6601_amd as t
    t.load()
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to the gpu-marked tests")
    return t


def _entries(rng, n, kind):
    m = rng.uniform(1.0, 2.0, n)
    if kind == "near one":
        return m * 2.0 ** rng.integers(-3, 4, n)
    if kind == "wide":
        return np.ldexp(m, rng.integers(-890, 1000, n))
    return np.ldexp(m, rng.integers(-1074, -900, n))  # tiny, subnormal ones among them


def _check_not_half_way(d):
    decimal.getcontext().prec = 60
    for v in d:
        r = decimal.Decimal(float(v)).sqrt()
        s = float(np.sqrt(v))
        ulp = decimal.Decimal(float(np.spacing(s)))
        off = (r - decimal.Decimal(s)) / ulp
        assert abs(abs(off) - decimal.Decimal("0.5")) > decimal.Decimal(2) ** -45


@pytest.mark.parametrize("kind", ["near one", "wide", "tiny"])
@pytest.mark.parametrize("n,nb", [(200, 64), (300, 128), (400, 192)])
def test_factor(tc, n, nb, kind):
    print("case n=%d nb=%d %s" % (n, nb, kind), flush=True)
    d = _entries(np.random.default_rng(n), n, kind)
    _check_not_half_way(d)
    A = torch.from_numpy(np.diag(d)).cuda()
    for inv in (False, True):
        W = A.clone()
        assert tc.factor_(W, nb, inv_trsm=inv) == 0
        L = np.tril(W.cpu().numpy().T)
        assert np.array_equal(np.diag(L), np.sqrt(d))
        assert not np.any(np.tril(L, -1))


@pytest.mark.parametrize("kind", ["near one", "wide", "tiny"])
def test_compact_batch(tc, kind):
    rng = np.random.default_rng(3)
    ns = [1, 16, 17, 32, 33, 100, 129, 300]
    ds = [_entries(rng, n, kind) for n in ns]
    for d in ds:
        _check_not_half_way(d)
    lda = [(n + 1) // 2 * 2 for n in ns]
    ao = np.concatenate([[0], np.cumsum([l * n for l, n in zip(lda, ns)])])
    bo = np.concatenate([[0], np.cumsum(ns)])
    flat = np.zeros(ao[-1])
    for d, n, l, o in zip(ds, ns, lda, ao):
        flat[o:o + l * n].reshape(n, l)[:, :n] = np.diag(d)
    A = torch.from_numpy(flat).cuda()
    B = torch.zeros(int(bo[-1]), dtype=torch.float64, device="cuda")
    info = tc.factor_solve_batched_(A, ao[:-1], lda, B, bo[:-1], ns, [(n + 15) // 16 * 16 for n in ns], 1)
    assert not np.any(info)
    got = A.cpu().numpy()
    for d, n, l, o in zip(ds, ns, lda, ao):
        L = got[o:o + l * n].reshape(n, l)[:, :n]
        assert np.array_equal(np.diag(L), np.sqrt(d))
