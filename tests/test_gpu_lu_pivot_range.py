"""Pivots near the ends of the FP64 range: the multipliers keep their accuracy while the
pivot's reciprocal is representable."""
import numpy as np
import pytest
import torch

from paper_2512_14193_amd import binding as B

pytestmark = pytest.mark.gpu


def middle(z, e):
    """z / 2^e in extended precision (exact)."""
    return np.ldexp(z.real.astype(np.longdouble), -e) + 1j * np.ldexp(z.imag.astype(np.longdouble), -e)


@pytest.mark.parametrize("n", [64, 400])
@pytest.mark.parametrize("e", [-1025, -1024, -1022, -1000, 1000, 1020, 1021, 1022])
def test_multipliers(n, e):
    """n / 2 blocks [[u, 0], [a, 1]] with 1.9 <= |u| / 2^e < 2.4 and a near u t, 0 < t < 1 (the
    components of 1/u stay below 2^1024 for the smallest e)."""
    print(f"[lu_pivot_range] n={n} e={e}", flush=True)
    rng = np.random.default_rng(n)
    m, ev, od = n // 2, np.arange(0, n, 2), np.arange(1, n, 2)
    u = np.ldexp(rng.uniform(1.7, 2.0, m), e) + 1j * np.ldexp(rng.uniform(0.9, 1.2, m), e)
    t = rng.uniform(0.2, 0.7, m)
    A = np.zeros((n, n), complex)
    A[ev, ev], A[od, ev], A[od, od] = u, u.real * t + 1j * (u.imag * t), 1.0
    W = B.fortran(torch.as_tensor(A).cuda())
    piv, info = B.zgetrf(W)
    torch.cuda.synchronize()
    lu, piv = W.cpu().numpy(), piv.cpu().numpy()
    assert info == 0 and np.array_equal(piv, np.arange(n))
    want = middle(A[od, ev], e) / middle(u, e)
    # 2^-53 for each of: the two of |u|^2, the reciprocal (2), its product, and the multiplier's
    # complex product (sqrt 5); and, where 1/u has denormal components, their rounding to a
    # multiple of 2^-1074: 2^-1074.5 against |1/u| >= 2^(-e - 1.3)
    bound = (5 + np.sqrt(5.0)) * 2.0 ** -53 + (2.0 ** (e - 1073.2) if e >= 1018 else 0.0)
    assert np.max(np.abs(lu[od, ev] - want) / np.abs(want)) <= bound
