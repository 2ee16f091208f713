"""Problems on one stream share the streams beside it: several alive at once, on the
default stream and on others, from several threads, destroyed in any order, give the
results of a problem alone."""
import threading

import numpy as np
import pytest
import torch

from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu


def solve(P, n, k0, rhs):
    P.assemble(I.star(n), I.Physics.from_wavenumbers(k0, 1.5 * k0))
    assert P.block_lu() == 0
    X = P.solve(rhs)
    P.sync()
    return X.cpu().numpy()


@pytest.mark.parametrize("n", [130, 700])
def test_alive_together(n):
    print(f"[side_streams] n={n}", flush=True)
    rhs = B.fortran(torch.as_tensor(I.probing_rhs(3 * n, 2, n)).cuda())
    ref = []
    for k in range(4):
        P = B.Problem(n)
        ref.append(solve(P, n, 3.0 + k, rhs))
        P.close()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    Ps = [B.Problem(n), B.Problem(n, stream=st), B.Problem(n), B.Problem(n, stream=st)]
    for order in ((0, 1, 2, 3), (2, 3), (3,)):  # the others are destroyed in between
        for k in order:
            assert np.array_equal(solve(Ps[k], n, 3.0 + k, rhs), ref[k])
        Ps[order[0]].close()
        if len(order) == 4:
            Ps[1].close()
    Ps[3].close()


def test_threads():
    n, rounds = 300, 4
    rhs = B.fortran(torch.as_tensor(I.probing_rhs(3 * n, 2, n)).cuda())
    P = B.Problem(n)
    ref = solve(P, n, 5.0, rhs)
    P.close()
    torch.cuda.synchronize()
    bad = []

    def work(own):
        st = torch.cuda.Stream() if own else None
        for _ in range(rounds):
            Q = B.Problem(n, stream=st) if own else B.Problem(n)
            if not np.array_equal(solve(Q, n, 5.0, rhs), ref):
                bad.append(own)
            Q.close()

    ts = [threading.Thread(target=work, args=(k % 2 == 1,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
