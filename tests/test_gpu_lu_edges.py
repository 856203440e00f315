"""The wavefront and workgroup LU where a zero pivot falls on the edges of their
panels and tiles, and the wavefront LU's arithmetic operation by operation.

A zero pivot makes what follows in that matrix meaningless (its reciprocal is NaN),
so the first zero step has to survive it, and the other matrices of the batch must
not notice.  The factors are those of an elimination that updates every entry with
one FMA per step, in order: U is compared for equality with math.h's fma on the
host, L with one product by a reciprocal that is good to a rounding or two (4 eps)."""
import ctypes

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


def first_zero_pivot(A):
    """Exact for totally unimodular matrices (every entry of the elimination is -1, 0 or 1)."""
    A = A.copy()
    for k in range(len(A)):
        p = k + int(np.argmax(np.abs(A[k:, k])))
        if A[p, k] == 0.0:
            return k + 1
        A[[k, p]] = A[[p, k]]
        A[k + 1:, k] /= A[k, k]
        A[k + 1:, k + 1:] -= np.outer(A[k + 1:, k], A[k, k + 1:])
    return 0


@pytest.mark.parametrize("n", [1, 5, 16, 17, 33, 55, 56, 64, 65, 80, 129, 151, 193, 256])
def test_zero_pivot_steps(chem, n):
    rng = np.random.default_rng(5000 + n)
    steps = sorted({s for s in (1, 2, 3, 4, 5, 8, 15, 16, 17, 32, 33, 48, 49, 63, 64, 65, 128, 129, 192, 193, n - 1, n)
                    if 1 <= s <= n})
    good = rng.standard_normal((n, n))
    mats, want = [good], [0]
    for s in steps:
        A = rng.standard_normal((n, n))
        A[:, s - 1] = 0.0  # stays exactly zero
        mats += [A, good]
        want += [s, 0]
    for row in range(1, n, max(1, n // 6)):  # two equal rows of a matrix of -1, 0 and 1 whose elimination is exact
        A = np.triu(np.ones((n, n)))[rng.permutation(n)]
        A[row] = A[row - 1]
        mats += [A, good]
        want += [first_zero_pivot(A), 0]
    A = torch.tensor(np.ascontiguousarray(mats), device=DEV)
    b = torch.ones((len(mats), n), dtype=torch.float64, device=DEV)
    LU, ipiv, info = (t.cpu().numpy() for t in chem.lu_factor(A))
    x, info2 = (t.cpu().numpy() for t in chem.lu_solve(A, b))
    np.testing.assert_array_equal(info, want)
    np.testing.assert_array_equal(info2, want)
    for m in (i for i, w in enumerate(want) if w == 0):
        np.testing.assert_array_equal(LU[m], LU[0])
        np.testing.assert_array_equal(ipiv[m], ipiv[0])
        np.testing.assert_array_equal(x[m], x[0])
    assert np.isfinite(LU[0]).all() and np.isfinite(x[0]).all()


@pytest.mark.parametrize("kind", ["random", "dominant"])
@pytest.mark.parametrize("n", [2, 5, 16, 17, 33, 55, 57, 64])
def test_one_fma_per_step(chem, n, kind):
    fma = ctypes.CDLL("libm.so.6").fma
    fma.restype, fma.argtypes = ctypes.c_double, [ctypes.c_double] * 3
    A = np.random.default_rng(5100 + n).standard_normal((n, n))
    if kind == "dominant":
        A += 3.0 * n * np.eye(n)
    LU, ipiv, info = (t[0].cpu().numpy() for t in chem.lu_factor(torch.tensor(A[None], device=DEV)))
    assert info == 0
    for k, p in enumerate(ipiv):
        A[[k, p]] = A[[p, k]]
    for i in range(n):
        for j in range(n):
            x = A[i, j]
            for k in range(min(i, j)):
                x = fma(-LU[i, k], LU[k, j], x)
            if i <= j:
                assert LU[i, j] == x, (i, j)
            else:
                assert abs(LU[i, j] - x / LU[j, j]) <= 4 * EPS * abs(LU[i, j]), (i, j)
