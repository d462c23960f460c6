"""Forces and potential of small groups (many more groups than wavefronts, which
are then not split): the same bits whatever the split, accelerations as without the
potential, and the potential of the direct sum within the walk's accuracy."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import _dev, _np, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gmax,n", [(1, 4099), (4, 12001), (16, 40009)])
def test_small_groups(nb, torch, gmax, n):
    _say("groups of up to", gmax, n)
    x, y, z, _, _, _, m = I.plummer(n, 47).f32()
    X, Y, Z, M = (_dev(torch, a) for a in (x, y, z, m))
    outs = []
    for split in (0, 1, 2, 4):
        ctx = nb.Context(nb.Params(group_max=gmax, leaf_max=gmax, walk_split=split), n_max=n)
        ctx.build_tree(X, Y, Z, M)
        a0 = ctx.calc_acc(None)
        acc, phi = ctx.calc_acc_pot(a0)
        outs.append(np.stack([_np(t) for t in (*acc, phi, *ctx.calc_acc(a0))]))
    np.testing.assert_array_equal(outs[0][:3], outs[0][4:])
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])
    t = torch.arange(0, n, 97, device="cuda")
    want = _np(ctx.direct64(X, Y, Z, M, t)[2])
    assert np.abs(outs[0][3][::97] / want - 1).max() <= 2e-2
