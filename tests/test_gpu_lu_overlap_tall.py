"""Orders between 2112 and 2560, whose product beside the panels is planned at the
product's own rate: the solution against the product formed first."""
import numpy as np
import pytest
import torch

from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2178, 2368, 2430])
def test_overlap_matches_product_first(n):
    print(f"[lu_overlap_tall] n={n}", flush=True)
    bnd, ph = I.star(n), I.Physics.from_wavenumbers(10.0, 20.0)
    Bh = B.fortran(torch.as_tensor(I.probing_rhs(3 * n, 2, n)).cuda())
    out = []
    for on in (True, False, True):
        P = B.Problem(n)
        P.set_lu_overlap(on)
        P.assemble(bnd, ph)
        assert P.block_lu() == 0
        out.append(P.solve(Bh))
        P.sync()
        P.close()
    a, b, c = (x.cpu().numpy() for x in out)
    assert np.array_equal(a, c)
    # other orders of the same sums: n eps times the growth of the solve, well below 1e-10
    assert np.max(np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)) < 1e-10
