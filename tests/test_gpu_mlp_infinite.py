"""The cost model on rows with an infinite feature (the library makes them: the
density of a group without mass is -inf) against the FP64 oracle: the units
saturate, so the prediction, the loss and every gradient but that of the
feature's own weights are finite (tolerances of test_gpu_costmodel.py)."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_costmodel import _dev, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [8, 16, 32, 64])
@pytest.mark.parametrize("col,bad", [(2, -np.inf), (1, np.inf), (0, np.inf)])
def test_infinite_feature(nb, torch, orc, H, col, bad):
    _say("mlp H", H, "feature", col, bad)
    rows = 40
    rng = np.random.default_rng(H)
    w = I.mlp_init(nb.mlp_nparams(H), orc.mlp_fan_in(H), 3)
    f = rng.standard_normal((rows, 4)).astype(np.float32)
    t = rng.standard_normal(rows).astype(np.float32)
    f[5, col] = bad
    ctx = nb.Context(nb.Params(), n_max=64)
    y = ctx.mlp_forward(H, _dev(torch, w), _dev(torch, f)).cpu().numpy()
    with np.errstate(all="ignore"):
        yo = orc.mlp_forward(w.astype(np.float64), f.astype(np.float64), hidden=H)
        lo, go = orc.mlp_grad(w.astype(np.float64), f.astype(np.float64), t.astype(np.float64),
                              hidden=H)
    ok = np.isfinite(yo)
    assert ok.sum() == rows - (col == 0)
    np.testing.assert_array_equal(y[~ok], yo[~ok])
    assert np.abs(y[ok] - yo[ok]).max() <= 1e-5 * np.abs(yo[ok]).max()
    if col == 0:
        return  # (an infinite prediction has no loss)
    g, loss = ctx.mlp_grad(H, _dev(torch, w), _dev(torch, f), _dev(torch, t))
    g = g.cpu().numpy()
    ok = np.isfinite(go)
    assert ok.sum() == len(w) - H  # all but the column's H weights of the first layer
    assert np.abs(g[ok] - go[ok]).max() <= 1e-4 * np.abs(go[ok]).max()
    assert abs(float(loss) - lo) <= 1e-5 * lo
