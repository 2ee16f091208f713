"""Which orders form their product in segments beside the panels: with the overlap on,
those up to about 2460 (so that a comparison with the product formed first compares two
paths), and none with it off."""
import pytest

from paper_2512_14193_amd import binding as B
from paper_2512_14193_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,taken", [(64, True), (130, True), (2112, True), (2178, True), (2368, True), (2430, True),
                                     (2496, False), (4096, False)])
def test_segments(n, taken):
    print(f"[lu_overlap_plan] n={n}", flush=True)
    P = B.Problem(n)
    P.assemble(I.star(n), I.Physics.from_wavenumbers(10.0, 20.0))
    for on in (True, False, True):
        P.set_lu_overlap(on)
        assert P.block_lu() == 0
        enabled, segments = P.lu_overlap_info()
        assert enabled == on and (segments > 0) == (on and taken), (on, segments)
        assert segments <= 10
    P.close()
