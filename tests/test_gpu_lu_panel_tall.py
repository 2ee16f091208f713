"""The panel kernel of 2049 to 2688 rows (seven wavefronts of rows, six rows a thread) at
its edges, single and batched, against LAPACK's pivots and the componentwise backward
error bound of Gaussian elimination."""
import numpy as np
import pytest
import scipy.linalg as sla
import torch

from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2240, 2241, 2687, 2688, 2689])
def test_pivots_and_backward_error(n):
    print(f"[lu_panel_tall] n={n}", flush=True)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    A[3, 0] = A[n - 1, 0] = 40.0  # equal candidates in the first and the last row slots: position decides
    W = B.fortran(torch.as_tensor(A).cuda())
    piv, info = B.zgetrf(W)
    torch.cuda.synchronize()
    lu, piv = W.cpu().numpy(), piv.cpu().numpy()
    assert info == 0 and piv[0] == 3
    assert np.array_equal(piv, sla.lu_factor(A)[1])
    P = A.copy()
    for c, p in enumerate(piv):
        P[[c, p]] = P[[p, c]]
    L, U = np.tril(lu, -1) + np.eye(n), np.triu(lu)
    # gamma = n eps with a factor 4 for complex arithmetic
    assert np.all(np.abs(P - L @ U) <= 4 * n * np.finfo(float).eps * (np.abs(L) @ np.abs(U)))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batched_equals_single(prec):
    n = 2178
    print(f"[lu_panel_tall] batch n={n} {prec}", flush=True)
    Ps = []
    for k in range(3):
        P = B.Problem(n, "mixed")
        if prec != "fp64":
            P.set_precision(prec, tol=1e-12)
        P.set_lu_overlap(False)
        P.assemble(I.star(n), I.Physics.from_wavenumbers(8.0, 12.0))
        Ps.append(P)
    assert Ps[0].block_lu() == 0
    assert B.block_lu_batch(Ps[1:]) == [0, 0]
    out = [P.copy_factors() for P in Ps]
    torch.cuda.synchronize()
    for lu, piv in out[1:]:
        assert torch.equal(lu, out[0][0]) and torch.equal(piv, out[0][1])
    for P in Ps:
        P.close()
