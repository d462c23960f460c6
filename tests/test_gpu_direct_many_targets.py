"""FP64 direct sums of many more targets than particles (a target may come up more
than once) against the FP64 oracle, at the edges of the small workgroups."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import _dev, _np, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 65, 512, 513])
def test_many_targets(nb, torch, orc, n):
    _say("direct64, particles", n)
    x, y, z, _, _, _, m = I.plummer(n, 8).f32()
    rng = np.random.default_rng(n)
    tgt = rng.integers(0, n, 4099).astype(np.int64)
    ask = tgt.copy()
    ask[[5, 4098]] = (-1, n)  # outside: sums nothing
    ctx = nb.Context(nb.Params(), n_max=16)
    acc, aabs, phi = ctx.direct64(*(_dev(torch, a) for a in (x, y, z, m)), _dev(torch, ask))
    ref = orc.direct(np.stack([x, y, z], 1).astype(np.float64), m, targets=tgt,
                     want_aabs=True, want_phi=True)
    for got, want in zip((acc, aabs, phi), ref):
        got, want = _np(got), want.copy()
        want[[5, 4098]] = 0.0
        assert np.abs(got - want).max() <= 1e-12 * max(np.abs(want).max(), 1e-300)
