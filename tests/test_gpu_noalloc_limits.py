"""The largest inputs of the allocation-free call: those it accepted before its
heavy groups had room of their own, and the size the header names for the default
parameters; bits as in the context path. Beyond it the call refuses."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import _dev, _np, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kw", [
    (81107, dict(leaf_max=1, waves_per_cu=4, frontier_cap=64, compensated=1)),
    (108575, dict(leaf_max=2, waves_per_cu=4, frontier_cap=128, compensated=1)),
    (133165, dict(leaf_max=4, waves_per_cu=8, frontier_cap=64, compensated=1)),
    (199876, dict(leaf_max=8, waves_per_cu=1, frontier_cap=64, compensated=1)),
    (58000, {})])
def test_accepted_sizes(nb, torch, n, kw):
    _say("allocation-free", n, kw)
    params = nb.Params(**kw)
    x, y, z, _, _, _, m = (_dev(torch, a) for a in I.plummer(n, 51).f32())
    ctx = nb.Context(params, n_max=n)
    ctx.build_tree(x, y, z, m)
    a0 = ctx.calc_acc(None)
    want = ctx.calc_acc(a0)
    out = tuple(torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(3))
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    nb.tree_forces_noalloc(params, x, y, z, m, a0, out, status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    for u, v in zip(out, want):
        np.testing.assert_array_equal(_np(u), _np(v))


def test_refused_size(nb, torch):
    x = torch.zeros(60000, dtype=torch.float32, device="cuda")
    with pytest.raises(nb.NbodyError) as e:
        nb.tree_forces_noalloc(nb.Params(), x, x, x, x, None, tuple(x.clone() for _ in range(3)))
    assert e.value.code == nb.NBODY_ENOMEM
