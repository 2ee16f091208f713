"""What a server factors together stays within its lanes' share of the panel workgroups
(16 each from N = 65 on), and more than eight lanes are served by eight."""
import pytest
import torch

from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu


def burst(s, n, count):
    bnd = I.star(n)
    geo = [torch.as_tensor(a, dtype=torch.float64, device="cuda").contiguous()
           for a in (bnd.x, bnd.dx, bnd.ddx, bnd.d3x)]
    reqs = []
    for i in range(count):
        rhs = B.fortran(torch.as_tensor(I.probing_rhs(3 * n, 4, i)).cuda())
        reqs.append((geo, I.Physics.from_wavenumbers(4.0 + 0.1 * i + 0.2j, 6.0), rhs, B.fortran_empty(3 * n, 4)))
    torch.cuda.synchronize()
    tickets = [s.submit(*r) for r in reqs]
    return reqs, [s.wait(t) for t in tickets]


@pytest.mark.parametrize("n,lanes,cmax,most", [(64, 4, 1024, 4), (128, 4, 1024, 2), (128, 2, 1024, 4),
                                               (512, 12, 512, 1), (1024, 4, 2048, 2)])
def test_batches_within_the_share(n, lanes, cmax, most):
    print(f"[serving_limits] n={n} lanes={lanes}", flush=True)
    s = B.Server(lanes=lanes, concurrent_max_n=cmax, batch_max=4)
    reqs, res = burst(s, n, 24)
    st = s.stats()
    s.close()
    assert all(r["status"] == 0 for r in res) and max(r["batched"] for r in res) <= most
    assert st["handles_created"] <= min(lanes, 8) * most
    # each result is that of the request alone (bitwise)
    P = B.Problem(n)
    P.set_lu_overlap(False)
    for (geo, ph, rhs, X) in reqs[::7]:
        P.assemble_device(geo, ph)
        P.block_lu()
        ref = P.solve(rhs)
        P.sync()
        assert torch.equal(X, ref)
    P.close()
