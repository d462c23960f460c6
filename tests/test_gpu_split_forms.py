"""The split walk of the compensated sum and of the potential: the same bits from
one, two or four wavefronts per group, and for the compensated sum from the
allocation-free call, which never splits it; compensated forces no further from
the direct double-precision sum than the rounding of the result and of the terms
(list sums at delta_acc = 0 hold every pair)."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import _dev, _np, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 65, 1000, 4161, 20011])
@pytest.mark.parametrize("comp", [0, 1])
def test_split_forms_give_the_same_bits(nb, torch, n, comp):
    _say("split forms", n, "compensated", comp)
    x, y, z, _, _, _, m = (_dev(torch, a) for a in I.plummer(n, 41).f32())
    outs = []
    for split in (1, 2, 4):
        ctx = nb.Context(nb.Params(walk_split=split, compensated=comp), n_max=n)
        ctx.build_tree(x, y, z, m)
        a0 = ctx.calc_acc(None)
        acc, phi = ctx.calc_acc_pot(a0)
        outs.append(np.stack([_np(t) for t in (*acc, phi, *ctx.calc_acc(a0))]))
    np.testing.assert_array_equal(outs[0][:3], outs[0][4:])
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])
    out = tuple(torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(3))
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    nb.tree_forces_noalloc(nb.Params(compensated=comp), x, y, z, m, tuple(a0), out, status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    np.testing.assert_array_equal(np.stack([_np(t) for t in out]), outs[0][:3])


@pytest.mark.parametrize("split", [1, 2])
def test_compensated_sum_stays_compensated(nb, torch, split):
    n = 3001
    x, y, z, _, _, _, m = I.plummer(n, 43).f32()
    ctx = nb.Context(nb.Params(walk_split=split, compensated=1, delta_acc=0.0), n_max=n)
    ctx.build_tree(*(_dev(torch, a) for a in (x, y, z, m)))
    a = np.stack([_np(t) for t in ctx.calc_acc(ctx.calc_acc(None))], 1).astype(np.float64)
    p = np.stack([x, y, z], 1).astype(np.float64)
    d = p[None] - p[:, None]
    f = m.astype(np.float64)[None] / ((d * d).sum(2) + 2.0 ** -14) ** 1.5
    want = (f[:, :, None] * d).sum(1)
    scale = (f * np.sqrt((d * d).sum(2))).sum(1)
    # each term: at most about 8 roundings of 2^-24; the sum adds one more
    assert (np.abs(a - want).max(1) <= 9 * 2.0 ** -24 * scale).all()
