"""Adaptive runs do not depend on the tile variant that a tuner picks by timing:
the error norm's partial sums are grouped alike in every variant, so error
norms, step sizes and states are the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
KW = dict(adaptive=True, dt0=0.002, rtol=1e-6, atol=1e-9)


def _fields(shape, seed):
    rng = np.random.default_rng(seed)
    return 0.16 + 0.02 * rng.standard_normal(shape), rng.uniform(0, 0.5, (3,) + shape)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,method", [((64, 64, 64), "ark436l"), ((96, 24, 40), "ark2"),
                                          ((168, 16, 56), "ark324l"), ((160, 8, 16), "ark436l"),
                                          ((504, 8, 16), "ark2")])
def test_single_grid_stage_tiles(params, shape, method, precision):
    from paper_2609_36100_amd import Solver
    print("[case] variant sums", shape, method, precision, flush=True)
    c, eta = _fields(shape, 21)
    out = []
    for variant in (0, 1):
        with Solver((shape[2], shape[1], shape[0]), params, method=method, precision=precision, **KW) as s:
            s.set_tuning(1, variant)
            s.set_state(c, eta)
            st = s.advance(0.02)
            out.append((s.kspace_to_numpy(s.get_state_hat()), st["err_last"], st["dt_last"], st["steps"]))
    assert out[0][1:] == out[1][1:]
    assert np.array_equal(out[0][0], out[1][0])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_ensemble_block_sizes(params, precision):
    from paper_2609_36100_amd import Ensemble
    print("[case] variant sums, ensemble", precision, flush=True)
    sizes = [48, 32, 128, 64, 96]
    fields = [_fields((n,) * 3, 30 + n) for n in sizes]
    out = []
    for threads in (128, 256):
        with Ensemble([dict(n=n, model=params, precision=precision, **KW) for n in sizes]) as E:
            for k in range(7):
                E.set_tuning(k, threads)
            for m, (c, eta) in enumerate(fields):
                E.set_state(m, c, eta)
            st = E.advance(0.02)
            out.append([(E.get_state_hat(m), st[m]["err_last"], st[m]["dt_last"], st[m]["steps"])
                        for m in range(len(sizes))])
    for a, b in zip(*out):
        assert a[1:] == b[1:]
        assert np.array_equal(a[0], b[0])
