"""The panel factorisation at the edges of its kernels (64, 512, 1024 and 2048 rows, one
row more, ragged last panels), against LAPACK's pivots and the componentwise backward
error bound of Gaussian elimination; equal candidates (the smallest position wins), zero
columns and columns of NaNs."""
import numpy as np
import pytest
import scipy.linalg as sla
import torch

from paper_2512_14193_amd import binding as B

pytestmark = pytest.mark.gpu


def factor(A):
    W = B.fortran(torch.as_tensor(A).cuda())
    piv, info = B.zgetrf(W)
    torch.cuda.synchronize()
    return W.cpu().numpy(), piv.cpu().numpy(), info


def interchange(A, piv):
    P = A.copy()
    for c, p in enumerate(piv):
        if p != c:
            P[[c, p]] = P[[p, c]]
    return P


@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 127, 512, 513, 577, 1024, 1025, 2048, 2049, 2113])
def test_pivots_and_backward_error(n):
    print(f"[lu_panel] n={n}", flush=True)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    lu, piv, info = factor(A)
    assert info == 0
    assert np.array_equal(piv, sla.lu_factor(A)[1])
    L, U = np.tril(lu, -1) + np.eye(n), np.triu(lu)
    # |P A - L U| <= gamma |L| |U| entry by entry, gamma = n eps with a factor 4 for complex arithmetic
    bound = 4 * n * np.finfo(float).eps * (np.abs(L) @ np.abs(U))
    assert np.all(np.abs(interchange(A, piv) - L @ U) <= bound)


@pytest.mark.parametrize("n", [40, 64, 200, 700, 1100, 2100])
def test_equal_candidates(n):
    """Rows of a lower triangle of ones in random order, with powers of two as column
    scales: every elimination step is exact and every remaining nonzero of a column has
    the same magnitude, so each pivot is decided by position alone."""
    print(f"[lu_panel] ties n={n}", flush=True)
    rng = np.random.default_rng(n)
    A = (np.tril(np.ones((n, n))) * 2.0 ** rng.integers(-3, 4, n))[rng.permutation(n)].astype(complex)
    lu, piv, info = factor(A)
    ref, order = A.copy(), []
    for c in range(n):
        p = c + int(np.argmax(np.abs(ref[c:, c].real) + np.abs(ref[c:, c].imag)))
        order.append(p)
        ref[[c, p]] = ref[[p, c]]
        ref[c + 1:, c] /= ref[c, c]
        ref[c + 1:, c + 1:] -= np.outer(ref[c + 1:, c], ref[c, c + 1:])
    assert info == 0
    assert np.array_equal(piv, order)
    assert np.array_equal(lu, ref)


@pytest.mark.parametrize("n", [50, 64, 600, 1500])
@pytest.mark.parametrize("value", [0.0, np.nan])
def test_column_without_pivot(n, value):
    """A zero column, or one of NaNs, below the diagonal of an identity: its diagonal row
    stays, the column is reported, and the panel that holds it has no other change above
    the diagonal of the column (later panels receive NaN multipliers in their updates)."""
    print(f"[lu_panel] n={n} column of {value}", flush=True)
    k = n // 3
    A = np.eye(n, dtype=complex)
    A[k:, k] = value
    lu, piv, info = factor(A)
    assert info == k + 1
    assert np.array_equal(piv, np.arange(n))
    panel = np.setdiff1d(np.arange(min(n, 64 * (k // 64 + 1))), [k])
    assert np.array_equal(lu[:k, panel], A[:k, panel])
    if value == 0.0:
        assert np.array_equal(lu, A)


@pytest.mark.parametrize("scale", [1e-290, 1e290])
def test_scaled_matrix(scale):
    """Powers of two commute with every rounding: the factors of a scaled matrix are the
    scaled factors."""
    n = 130
    rng = np.random.default_rng(7)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    s = 2.0 ** round(np.log2(scale))
    lu, piv, info = factor(A * s)
    ref, pr, _ = factor(A)
    assert info == 0 and np.array_equal(piv, pr)
    assert np.array_equal(np.tril(lu, -1), np.tril(ref, -1))
    assert np.array_equal(np.triu(lu), np.triu(ref) * s)
