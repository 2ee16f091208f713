"""Factorisations captured into HIP graphs, several problems alive on one stream: with the
overlap on they form U33 first, bitwise as with it off, on every replay and beside the
eager (overlapped) calls of other problems."""
import pytest
import torch

from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [130, 700])
def test_replays_equal_product_first(n):
    print(f"[lu_capture] n={n}", flush=True)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        rhs = B.fortran(torch.as_tensor(I.probing_rhs(3 * n, 9, n)).cuda())
        Ps, Xs, first, eager = [], [], [], []
        for k in range(3):
            P = B.Problem(n, stream=st)
            P.assemble(I.star(n), I.Physics.from_wavenumbers(4.0 + k + 0.2j, 7.0))
            for on, out in ((False, first), (True, eager)):
                P.set_lu_overlap(on)
                P.block_lu()
                out.append(P.solve(rhs).clone())
            assert P.lu_overlap_info()[1] > 0
            Ps.append(P)
            Xs.append(B.fortran_empty(3 * n, 9))
        st.synchronize()
        graphs = []
        for P, X in list(zip(Ps, Xs))[:2]:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
                P.block_lu(sync=False)
                P.solve(rhs, X)
            assert P.lu_overlap_info()[1] == 0
            graphs.append(g)
        for rep in range(4):
            for X in Xs:
                X.zero_()
            graphs[0].replay()
            graphs[1].replay()
            Ps[2].block_lu(sync=False)
            Ps[2].solve(rhs, Xs[2])
            if rep % 2:
                st.synchronize()
            graphs[0].replay()
            st.synchronize()
            assert torch.equal(Xs[0], first[0]) and torch.equal(Xs[1], first[1]) and torch.equal(Xs[2], eager[2])
        Ps[1].block_lu()  # eager again
        assert Ps[1].lu_overlap_info()[1] > 0 and torch.equal(Ps[1].solve(rhs), eager[1])
        st.synchronize()
        del graphs
        for P in Ps:
            P.close()
