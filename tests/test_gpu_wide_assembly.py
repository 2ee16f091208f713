"""Assembly in the wide domain on both sides of the order up to which each workgroup makes
its own tables (1200 nodes), and at the smallest orders, against the oracle; the limit
|k| r < 6 is reported on either side."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu
K0, K1 = 1.3 - 1.68j, 2.6 - 3.36j  # |k1| r < 4.3 on the disk of radius 1/2


@pytest.mark.parametrize("form", ["mixed", "ordinary"])
@pytest.mark.parametrize("n", [8, 34, 1200, 1202])
def test_blocks(n, form):
    print(f"[wide_assembly] n={n} {form}", flush=True)
    bnd, ph = I.disk(n, 0.5), I.Physics.from_wavenumbers(K0, K1)
    P = B.Problem(n, form)
    P.assemble(bnd, ph)
    out = P.copy_blocks()
    P.sync()
    if form == "mixed":
        M = O.build_mixed(bnd, ph)
        top, bot = (x.cpu().numpy() for x in out)
        pairs = [(top[:n], M[:n, 2 * n:]), (top[n:], M[n:2 * n, 2 * n:]), (bot, M[2 * n:, :2 * n])]
    else:
        pairs = [(out.cpu().numpy(), O.build_ordinary(bnd, ph))]
    for got, ref in pairs:
        # a few ulps of the Hankel and Bessel values, which the logarithmic split scales by up to
        # the largest entry
        assert np.max(np.abs(got - ref)) <= 1e-13 * np.max(np.abs(ref))
        assert np.linalg.norm(got - ref) <= 1e-13 * np.linalg.norm(ref)
    P.close()


@pytest.mark.parametrize("n", [64, 1202])
def test_limit(n):
    print(f"[wide_assembly] limit n={n}", flush=True)
    P = B.Problem(n, "mixed")
    P.assemble(I.disk(n, 0.5), I.Physics.from_wavenumbers(K0, 4.0 - 5.0j))  # |k1| r up to 6.4
    with pytest.raises(B.BMError) as e:
        P.sync()
    assert e.value.code == B.BM_E_DOMAIN
    P.assemble(I.disk(n, 0.5), I.Physics.from_wavenumbers(K0, K1))
    P.sync()
    P.close()
