"""The tiled wavefront LU at the edges of its four-column panels and 16-column
tiles, against a step-by-step elimination in plain numpy.

The rank-4 updates on the matrix cores repeat the elimination's operations in
the same order, each product and sum with one rounding (an FMA), so the pivots
must be equal and the factors agree to the difference between an FMA and a
separate multiplication and addition: at most n roundings of intermediate
values, each up to |l| max |u| <= growth * max |A|, with |l| <= 1.  The
tolerance is 4 n eps max |LU| per entry.  Row orders that leave the diagonal tile
(random matrices, reversed rows) and natural order (a dominant diagonal) take
different branches of the update."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def chem():
    from paper_2105_12070_amd import chem as c
    assert torch.cuda.is_available()
    return c


def getrf(A):
    A = A.copy()
    n = A.shape[0]
    piv = np.zeros(n, np.int32)
    for k in range(n):
        p = k + int(np.argmax(np.abs(A[k:, k])))
        piv[k] = p
        A[[k, p]] = A[[p, k]]
        A[k + 1:, k] /= A[k, k]
        A[k + 1:, k + 1:] -= np.outer(A[k + 1:, k], A[k, k + 1:])
    return A, piv


def matrices(n, kind, rng):
    A = rng.standard_normal((5, n, n))
    if kind == "dominant":
        A += 3.0 * n * np.eye(n)
    elif kind == "reversed":
        A = (A + 3.0 * n * np.eye(n))[:, ::-1].copy()
    return A


@pytest.mark.parametrize("kind", ["random", "dominant", "reversed"])
@pytest.mark.parametrize("n", [1, 2, 4, 5, 15, 16, 17, 20, 31, 32, 33, 36, 47, 48, 49, 52, 53, 55, 56, 57, 60, 61, 63, 64])
def test_panels_match_elimination(chem, n, kind):
    A = matrices(n, kind, np.random.default_rng(900 + n))
    LU, ipiv, info = chem.lu_factor(torch.tensor(A, device=DEV))
    b = np.random.default_rng(n).standard_normal((5, n))
    x, info2 = chem.lu_solve(torch.tensor(A, device=DEV), torch.tensor(b, device=DEV))
    LU, ipiv, x = LU.cpu().numpy(), ipiv.cpu().numpy(), x.cpu().numpy()
    assert np.all(info.cpu().numpy() == 0) and np.all(info2.cpu().numpy() == 0)
    for m in range(5):
        ref, piv = getrf(A[m])
        np.testing.assert_array_equal(ipiv[m], piv)
        assert np.abs(LU[m] - ref).max() <= 4 * n * EPS * np.abs(ref).max()
        # the solve's residual: backward error of a pivoted LU solve
        res = np.abs(A[m] @ x[m] - b[m]).max()
        assert res <= 10 * n * EPS * (np.abs(A[m]).sum(1).max() * np.abs(x[m]).max() + np.abs(b[m]).max())


@pytest.mark.parametrize("kind", ["random", "dominant", "reversed"])
@pytest.mark.parametrize("n", [65, 80, 127, 128, 129, 143, 160, 161, 192, 193, 208, 255, 256])
def test_workgroup_panels_backward_error(chem, n, kind):
    """Above 64: sizes at the edges of the panel's register slots (64, 128, 192 rows) and of its 16 columns, with many,
    all and no interchanges.  |P A - L U| <= gamma_n |L| |U| entry by entry holds for any order of the elimination's
    sums (Higham, Accuracy and Stability, Theorem 9.3); the multiplication by a rounded reciprocal and the residual's
    own sums add as much again: (2 n + 8) eps |L| |U|."""
    A = matrices(n, kind, np.random.default_rng(1900 + n))
    LU, ipiv, info = chem.lu_factor(torch.tensor(A, device=DEV))
    LU, ipiv = LU.cpu().numpy(), ipiv.cpu().numpy()
    assert np.all(info.cpu().numpy() == 0)
    for m in range(5):
        np.testing.assert_array_equal(ipiv[m], getrf(A[m])[1])
        PA = A[m].copy()
        for k, p in enumerate(ipiv[m]):
            PA[[k, p]] = PA[[p, k]]
        L, U = np.tril(LU[m], -1) + np.eye(n), np.triu(LU[m])
        assert np.all(np.abs(PA - L @ U) <= (2 * n + 8) * EPS * (np.abs(L) @ np.abs(U)))
