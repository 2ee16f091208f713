"""The complex64 LU's trailing update (64 x 64 tiles, depth slices of 16) at orders
around its tiles' edges, against the oracle's Schur complement and against the
batched factorisation."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [66, 128, 130, 190, 192, 194, 256, 258, 322])
def test_factors_reproduce_the_matrix(n):
    """|L U - P U33| / |U33| at FP32 rounding: 2e-6 is the bound that larger orders
    are held to; one wrong row, column or depth slice of an update is of order
    1 / sqrt(n)."""
    print(f"[update32] n={n}", flush=True)
    bnd, ph = I.star(n), I.Physics.from_wavenumbers(3.0, 4.5)
    Ps = [B.Problem(n, "mixed") for _ in range(2)]
    for P in Ps:
        P.set_precision("mixed", tol=1e-12, max_iter=10)
        P.assemble(bnd, ph)
    assert Ps[0].block_lu() == 0
    P1 = [Ps[1]]
    assert all(i == 0 for i in B.block_lu_batch(P1))
    out = []
    for P in Ps:
        lu, piv = P.copy_factors()
        torch.cuda.synchronize()
        out.append((lu.cpu().numpy(), piv.cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    lu, piv = out[0]
    A = O.build_mixed(bnd, ph)
    u33 = A[2 * n:, 2 * n:] - A[2 * n:, :n] @ A[:n, 2 * n:] - A[2 * n:, n:2 * n] @ A[n:2 * n, 2 * n:]
    pu = u33.copy()
    for i in range(n):
        pu[[i, piv[i]]] = pu[[piv[i], i]]
    err = np.linalg.norm((np.tril(lu, -1) + np.eye(n)) @ np.triu(lu) - pu) / np.linalg.norm(u33)
    assert err < 2e-6, err
    for P in Ps:
        P.close()
