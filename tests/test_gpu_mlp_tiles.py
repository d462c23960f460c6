"""The cost model's matrix-core kernels at the edges of their 32-row tiles and
32-unit blocks against the FP64 oracle (tolerances of test_gpu_costmodel.py),
and training in one call against a gradient and an Adam call per step."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_costmodel import _dev, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _rows(n, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((n, 4)).astype(np.float32),
            rng.standard_normal(n).astype(np.float32))


@pytest.mark.parametrize("H", [8, 16, 32, 64])
@pytest.mark.parametrize("rows", [1, 31, 32, 33, 129, 33000])
def test_mlp_tile_edges(nb, torch, orc, H, rows):
    ctx = nb.Context(nb.Params(), n_max=64)
    w = I.mlp_init(nb.mlp_nparams(H), orc.mlp_fan_in(H), 3)
    f, t = _rows(rows, rows + H)
    W, F, T = _dev(torch, w), _dev(torch, f), _dev(torch, t)
    y = ctx.mlp_forward(H, W, F).cpu().numpy()
    yo = orc.mlp_forward(w.astype(np.float64), f.astype(np.float64), hidden=H)
    assert np.abs(y - yo).max() <= 1e-5 * np.abs(yo).max()
    g, loss = ctx.mlp_grad(H, W, F, T)
    lo, go = orc.mlp_grad(w.astype(np.float64), f.astype(np.float64), t.astype(np.float64),
                          hidden=H)
    err = np.abs(g.cpu().numpy() - go).max() / np.abs(go).max()
    _say("mlp H %d rows %d: gradient off by %.2g of its largest entry" % (H, rows, err))
    assert err <= 1e-4
    assert abs(float(loss) - lo) <= 1e-5 * lo


@pytest.mark.parametrize("H", [8, 64])
def test_training_equals_single_steps(nb, torch, H):
    ctx = nb.Context(nb.Params(), n_max=64)
    w0 = I.mlp_init(nb.mlp_nparams(H), nb.mlp_fan_in(H), 4)
    f, t = _rows(777, 5)
    F, T = _dev(torch, f), _dev(torch, t)
    W = _dev(torch, w0)
    losses = ctx.train_cost_model(H, W, F, T, 5, 1e-2)
    one = _dev(torch, w0)
    first = _dev(torch, w0)
    ctx.train_cost_model(H, first, F, T, 1, 1e-2)  # (sets the standardisation)
    one[:8] = first[:8]
    m, v = torch.zeros_like(one), torch.zeros_like(one)
    for k in range(5):
        g, loss = ctx.mlp_grad(H, one, F, T)
        assert float(loss) == losses[k]
        ctx.mlp_adam(one, g, m, v, k + 1, 1e-2)
    np.testing.assert_array_equal(one.cpu().numpy(), W.cpu().numpy())
