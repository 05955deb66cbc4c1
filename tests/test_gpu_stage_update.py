"""Stage and update passes (every F^I formed again from the state and the
explicit derivatives, one field per work-group) at the line lengths whose
work-groups are not whole wavefronts, for every pair, both precisions and both
splits, against the oracle's steps: 1e-10 relative L2 of the whole state in
FP64 (the stated target), 1e-5 in the mixed form (its stated bound on states
after a few steps)."""
import numpy as np
import pytest

from oracle import ark as oark
from oracle import model as om

pytestmark = pytest.mark.gpu
TABLES = {"imex_euler": oark.imex_euler, "ark2": oark.ark2, "ark324l": oark.ark324l2sa, "ark436l": oark.ark436l2sa}


@pytest.mark.parametrize("method", list(TABLES))
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("mixed", 1e-5)])
@pytest.mark.parametrize("shape,bulk", [((8, 16, 24), 1), ((24, 8, 40), 0), ((56, 24, 8), 1), ((168, 8, 16), 0)])
def test_steps_match_oracle(params, shape, bulk, precision, tol, method):
    from paper_2609_36100_amd import Solver
    print("[case] stage", shape, bulk, precision, method, flush=True)
    prm = dict(params, implicit_bulk_c=bulk)
    rng = np.random.default_rng(5)
    c = 0.16 + 0.02 * rng.standard_normal(shape)
    eta = rng.uniform(0, 1, (3,) + shape)
    mdl = om.Model(shape, prm)
    y = om.to_kspace(c, eta)
    with Solver((shape[2], shape[1], shape[0]), prm, method=method, precision=precision, dt0=0.02) as s:
        s.set_state_hat(s.kspace_from_numpy(y))
        for variant in (0, 1):
            s.set_tuning(1, variant)
            y, _, _ = oark.ark_step(y, 0.02, TABLES[method](), mdl.f_explicit, mdl.implicit_symbol())
            ok, _, _ = s.step(0.02)
            assert ok
            g = s.kspace_to_numpy(s.get_state_hat())
            rel = np.linalg.norm(g - y) / np.linalg.norm(y)
            assert rel < tol, (variant, rel)
