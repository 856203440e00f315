"""LU of matrices that hold NaN or Inf: what is reported, and which entries of the
factors stay finite.

The reference is the step-by-step elimination in numpy, in which a value reaches
only the entries that the algorithm updates: rows not yet chosen, columns right
of the pivot.  An entry that the reference holds finite has to be finite in the
factors too, and to agree to 4 n eps max |LU| (at most n roundings of values up to
max |LU|, an FMA against a separate multiplication and addition)."""
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


def getrf_passing_nan(A):
    """The workgroup LU's rules (n > 64): padded with unit rows to a multiple of 16; the pivot is the largest |a| that
    is not NaN, the first of them, and the current row where all are NaN; the reciprocal of an Inf pivot is NaN."""
    n = A.shape[0]
    m = (n + 15) // 16 * 16
    M = np.eye(m)
    M[:n, :n] = A
    piv, info = np.zeros(m, np.int32), 0
    with np.errstate(all="ignore"):
        for k in range(m):
            c = np.abs(M[k:, k])
            p = k if np.isnan(c).all() else k + int(np.nanargmax(c))
            if M[p, k] == 0.0:
                info = info or k + 1
                p = k
            piv[k] = p
            M[[k, p]] = M[[p, k]]
            r = 0.0 if info == k + 1 else np.nan if np.isinf(M[k, k]) else 1.0 / M[k, k]
            M[k + 1:, k] *= r
            M[k + 1:, k + 1:] -= np.outer(M[k + 1:, k], M[k, k + 1:])
    return M[:n, :n], piv[:n], info


def spoiled(n, kind):
    A = np.random.default_rng(3100 + n).standard_normal((n, n)) + 3.0 * n * np.eye(n)  # row k is the pivot of step k
    if kind == "nan_entry":
        A[n // 2, n // 2] = np.nan
    elif kind == "nan_first":
        A[0, 0] = np.nan
    elif kind == "nan_row":
        A[n // 3] = np.nan
    elif kind == "nan_zero_column":
        A[:, n - 2], A[n - 1, n - 2] = 0.0, np.nan
    elif kind == "inf_last_column":
        A[n - 5, n - 1] = np.inf
    elif kind == "inf_in_panel":
        A[5, 14] = np.inf
    return A


KINDS = ["nan_entry", "nan_first", "nan_row", "nan_zero_column", "inf_last_column", "inf_in_panel"]


# the panel in LDS (above 192 rows) divides by an Inf pivot and gets 0
@pytest.mark.parametrize("n,kind", [(n, k) for n in (65, 80, 128, 129, 151, 192, 193, 256) for k in KINDS
                                    if n <= 192 or k != "inf_in_panel"])
def test_workgroup_lu(chem, n, kind):
    """65 to 192 rows: 2 and 3 register slots of the panel, then 1; above 192 the first panels are factored in LDS.
    A matrix without NaN or Inf on either side must not notice."""
    A = spoiled(n, kind)
    good = np.random.default_rng(3200 + n).standard_normal((n, n))
    B = np.stack([good, A, good])
    LU, ipiv, info = (t.cpu().numpy() for t in chem.lu_factor(torch.tensor(B, device=DEV)))
    x, info2 = (t.cpu().numpy() for t in chem.lu_solve(torch.tensor(B, device=DEV),
                                                       torch.ones((3, n), dtype=torch.float64, device=DEV)))
    ref, piv, want = getrf_passing_nan(A)
    np.testing.assert_array_equal(info, [0, want, 0])
    np.testing.assert_array_equal(info2, [0, want, 0])
    np.testing.assert_array_equal(LU[0], LU[2])
    np.testing.assert_array_equal(x[0], x[2])
    assert np.isfinite(LU[0]).all() and np.isfinite(x[0]).all()
    if want:
        return
    fin = np.isfinite(ref)
    np.testing.assert_array_equal(ipiv[1], piv)
    assert np.isfinite(LU[1][fin]).all()
    assert np.abs(LU[1][fin] - ref[fin]).max() <= 4 * n * EPS * np.abs(ref[fin]).max()


def getrf_wave(A):
    """The wavefront LU's rules (n <= 64): NaN is the largest of all, the first of them; the reciprocal of a pivot that
    is Inf, NaN or below the normal range is NaN; every row takes part in the updates, those already chosen with a
    multiplier of 0."""
    M, n = A.copy(), A.shape[0]
    piv = np.zeros(n, np.int32)
    with np.errstate(all="ignore"):
        for k in range(n):
            p = k + int(np.argmax(np.abs(M[k:, k])))  # numpy's argmax takes the first NaN
            piv[k] = p
            M[[k, p]] = M[[p, k]]
            a = abs(M[k, k])
            M[k + 1:, k] *= 1.0 / M[k, k] if np.finfo(np.float64).tiny <= a < np.inf else np.nan
            M[k + 1:, k + 1:] -= np.outer(M[k + 1:, k], M[k, k + 1:])
            M[:k + 1, k + 1:] -= np.outer(np.zeros(k + 1), M[k, k + 1:])
    return M, piv


def spoiled_wave(n, kind):
    A = np.random.default_rng(3300 + n).standard_normal((n, n))
    if kind.endswith("dominant"):
        A += 3.0 * n * np.eye(n)
    i = n // 2
    if kind.startswith("nan_entry"):
        A[i, i] = np.nan
    elif kind.startswith("inf_entry"):
        A[i, i] = np.inf
    elif kind.startswith("subnormal_column"):
        A[:, i] *= 1e-316
    elif kind.startswith("nan_late"):
        A[:, n - 1] = np.nan
    return A


@pytest.mark.parametrize("kind", [a + b for a in ("nan_entry", "inf_entry", "subnormal_column", "nan_late")
                                  for b in ("", "_dominant")])
@pytest.mark.parametrize("n", [2, 5, 16, 17, 33, 55, 56, 57, 64])
def test_wavefront_factors(chem, n, kind):
    """Columns finished before the NaN arose stay as they are, also within the 16-column tile that it arises in."""
    A = spoiled_wave(n, kind)
    good = np.random.default_rng(3400 + n).standard_normal((n, n))
    LU, ipiv, info = (t.cpu().numpy() for t in chem.lu_factor(torch.tensor(np.stack([good, A, good]), device=DEV)))
    ref, piv = getrf_wave(A)
    np.testing.assert_array_equal(info, 0)
    np.testing.assert_array_equal(LU[0], LU[2])
    assert np.isfinite(LU[0]).all()
    fin = np.isfinite(ref)
    first_nan = int(np.argmax(np.isnan(ref).any(0))) if np.isnan(ref).any() else n
    np.testing.assert_array_equal(ipiv[1][:first_nan + 1], piv[:first_nan + 1])
    assert np.isfinite(LU[1][fin]).all()
    assert np.abs(LU[1][fin] - ref[fin]).max() <= 4 * n * EPS * np.abs(ref[fin]).max()
