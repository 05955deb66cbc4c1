"""The elastic iteration on strains that are not finite: a change that is NaN is
not at most the tolerance, so the iteration takes all its updates (as the
oracle's, whose largest change is NaN too) and does not report convergence after
the first one."""
import numpy as np
import pytest

from oracle import elastic_inhom as ei
from oracle import model as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("max_iter", [1, 5])
def test_nan_strain_does_not_converge(params, bad, max_iter):
    import warnings
    from paper_2609_36100_amd import Solver
    print("[case] inhom", bad, max_iter, flush=True)
    p = dict(params)
    p.update(C11p=1.5 * p["C11"], C12p=1.5 * p["C12"], C44p=1.5 * p["C44"], el_tol=1e-6, el_max_iter=max_iter)
    n = 16
    rng = np.random.default_rng(4)
    eta = rng.uniform(0, 1, (3, n, n, n))
    y = om.to_kspace(0.16 + 0.01 * rng.standard_normal((n, n, n)), eta)
    y[1, 2, 3, 1] = bad
    m = ei.InhomModel((n, n, n), p)
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        m.f_explicit(y)
    with Solver(n, p) as s:
        _, fE = s.rhs(s.kspace_from_numpy(y))
        assert np.isnan(s.kspace_to_numpy(fE)[1:]).any()
        assert s.stats()["el_last"] == m.last_iterations == max_iter
