"""Surrogate kernels at the edges of their tiles: widths and hidden sizes that do
not fill 32-channel tiles, the widths on either side of the fused projection
(32), channel counts that four or eight do not divide, grids whose x lines a
wave does not fill.  Forward output and loss at 3e-2 and every gradient at 3e-2
relative L2 against the FP64 oracle (the BF16 network's stated bound)."""
import numpy as np
import pytest

from oracle import fno as of

pytestmark = pytest.mark.gpu
BOUND = 3e-2


@pytest.mark.parametrize("n,w,m,L,h,cin,cout",
                         [(8, 36, 2, 2, 72, 4, 4), (32, 24, 4, 2, 96, 4, 4), (32, 20, 4, 2, 40, 5, 3),
                          (40, 32, 4, 1, 128, 4, 4), (16, 4, 2, 1, 8, 1, 1), (8, 128, 2, 1, 128, 8, 8)])
def test_forward_and_gradients(n, w, m, L, h, cin, cout):
    import torch
    from paper_2609_36100_amd import FNO
    print("[case] fno shapes", n, w, m, L, h, cin, cout, flush=True)
    net = of.FNO(n, width=w, modes=m, layers=L, cin=cin, cout=cout, hidden=h)
    rng = np.random.default_rng(9)
    p = net.init_params(seed=3)
    for k in p:
        if k[0] in "bc":
            p[k] = 0.1 * rng.standard_normal(p[k].shape)
    to_bf = lambda a: torch.from_numpy(np.asarray(a, np.float32)).to(torch.bfloat16).to(torch.float64).numpy()
    p = {k: to_bf(v) for k, v in p.items()}
    x = rng.uniform(-1, 1, (n, n, n, cin))
    x = to_bf(x - x.mean(axis=(0, 1, 2)))
    tgt = rng.standard_normal((n, n, n, cout)) * 0.5
    out, tape = net.forward(p, x, keep=True)
    loss, dout = of.mse_loss(out, tgt)
    g = net.backward(p, tape, dout)
    xt = torch.from_numpy(np.ascontiguousarray(np.moveaxis(x, -1, 0))).float().cuda()
    yt = torch.zeros_like(xt)
    yt[:cout] = xt[:cout] + torch.from_numpy(np.ascontiguousarray(np.moveaxis(tgt, -1, 0))).float().cuda()
    with FNO(n, width=w, modes=m, layers=L, hidden=h, cin=cin, cout=cout) as f:
        f.set_params(np.concatenate([p[k].ravel() for k in net.param_shapes()]).astype(np.float32))
        gout = f.forward(xt).cpu().numpy().reshape(n, n, n, cout)
        f.zero_grad()
        gl = f.grad(xt, yt)
        flat = f.get_grad().astype(np.float64)
    assert np.linalg.norm(gout - out) < BOUND * np.linalg.norm(out)
    assert abs(gl - loss) < BOUND * loss
    at = 0
    for k, s in net.param_shapes().items():
        a = flat[at:at + int(np.prod(s))].reshape(s)
        at += a.size
        assert np.linalg.norm(a - g[k]) < BOUND * np.linalg.norm(g[k]) + 1e-30, k
