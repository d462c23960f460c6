"""Which groups are walked in parts: a_old a thousand times too small (every list
long, no group cut but those with scattered members), and a_old whose size differs
from particle to particle (every group cut, more parts than there are slots, so
that most groups' sums are made one part after the other). Lists and entry hashes
equal the oracle's, forces hold the tree-parity rule, and the bits are the same from
any stack size, split and wavefront count and from the allocation-free call."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import (_assert_rule, _compare_walk, _dev, _np, _ref, _run, _say,  # noqa: F401
                             nb, torch)

pytestmark = pytest.mark.gpu


def _a_old(kind, acc, rng):
    if kind == "small":
        return (acc * 1e-3).astype(np.float32)
    return (acc * 10.0 ** rng.uniform(-6, -4, (len(acc), 1))).astype(np.float32)


@pytest.mark.parametrize("comp", [0, 1])
@pytest.mark.parametrize("kind,n", [("small", 9000), ("uneven", 4097), ("uneven", 20011)])
def test_long_lists_match_oracle(nb, torch, orc, kind, n, comp):
    _say("a_old", kind, n, "compensated", comp)
    x, y, z, _, _, _, m = I.galaxy(n, 17).f32()
    params = nb.Params(compensated=comp)
    a_old = _a_old(kind, _ref(orc, x, y, z, m, params).acc, np.random.default_rng(n))
    ctx, acc = _run(nb, torch, x, y, z, m, params, a_old=a_old)
    ref = _ref(orc, x, y, z, m, params, a_old)
    assert ref.gentries.min() > 2048
    e, et = _compare_walk(nb, ctx, ref, acc, np.stack([x, y, z], 1), m, 2.0 ** -7)
    _assert_rule(e, et)


@pytest.mark.parametrize("kind", ["small", "uneven"])
def test_long_lists_do_not_depend_on_the_walk(nb, torch, orc, kind):
    n = 20011
    x, y, z, _, _, _, m = I.galaxy(n, 17).f32()
    a_old = _a_old(kind, _ref(orc, x, y, z, m, nb.Params()).acc, np.random.default_rng(n))
    outs = []
    for fc, split, waves in ((0, 0, 32), (64, 2, 4), (512, 4, 12), (0, 1, 1)):
        outs.append(_run(nb, torch, x, y, z, m,
                         nb.Params(frontier_cap=fc, walk_split=split, waves_per_cu=waves),
                         a_old=a_old)[1])
    out = tuple(torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(3))
    nb.tree_forces_noalloc(nb.Params(), *(_dev(torch, a) for a in (x, y, z, m)),
                           tuple(_dev(torch, a_old[:, k]) for k in range(3)), out)
    outs.append(np.stack([_np(t) for t in out], 1))
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])
