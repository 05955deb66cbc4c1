"""Plane passes (y and x transforms of a plane in one kernel, nx == ny small):
the right-hand side on every plane size they take, with few and many planes,
against the oracle, on a state whose kx = 0 and Nyquist columns are not
Hermitian (the c2r drops those imaginary parts): 1e-10 relative L2 per field.
The composition's f^E there is compared on Hermitian states only: the oracle
forms it from the real field minus the implicit part of y itself, the library
as 2 W M (c_p - c_m) k^2 H~, and the two are equal only where y is the transform
of a real field."""
import numpy as np
import pytest

from oracle import model as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nz", [(8, 16), (16, 8), (24, 24), (32, 8), (48, 16), (64, 8), (64, 64)])
@pytest.mark.parametrize("hermitian", [True, False])
def test_rhs_on_planes(params, n, nz, hermitian):
    from paper_2609_36100_amd import Solver
    print("[case] plane", n, nz, hermitian, flush=True)
    rng = np.random.default_rng(n + nz)
    shape = (nz, n, n)
    y = om.to_kspace(0.16 + 0.02 * rng.standard_normal(shape), rng.uniform(0, 1, (3,) + shape))
    if not hermitian:
        for k in (0, n // 2):
            z = rng.standard_normal((4, nz, n)) + 1j * rng.standard_normal((4, nz, n))
            y[..., k] += 0.05 * np.abs(y[..., k]).mean() * z
    FI, FE = om.Model(shape, params).rhs(y)
    with Solver((n, n, nz), params) as s:
        fI, fE = s.rhs(s.kspace_from_numpy(y))
        fI, fE = s.kspace_to_numpy(fI), s.kspace_to_numpy(fE)
    for f in range(4):
        assert np.linalg.norm(fI[f] - FI[f]) <= 1e-10 * np.linalg.norm(FI[f])
        if f == 0 and not hermitian:
            continue
        assert np.linalg.norm(fE[f] - FE[f]) <= 1e-10 * np.linalg.norm(FE[f]), f
