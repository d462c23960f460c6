"""Groups walked in parts that meet an over-full leaf (6000 particles at one point),
which their parts take in slices; with an uneven a_old every group is cut and there
are more parts than slots. Lists and entry hashes equal the oracle's, compensated
forces hold the tree-parity rule, plain ones the bound of their sums' roundings, and
the bits are the same from any stack size, split and wavefront
count and from the allocation-free call."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_heavy_rule import _a_old
from test_gpu_parity import (_assert_rule, _compare_walk, _dev, _np, _ref, _run, _say,  # noqa: F401
                             nb, torch)

pytestmark = pytest.mark.gpu
N = 20011


def _input(orc, uneven):
    x, y, z, _, _, _, m = I.plummer(N, 17).f32()
    for a in (x, y, z):
        a[100:6100] = a[100] * np.float32(0.125)
    a_old = _ref(orc, x, y, z, m, _params()).acc.astype(np.float32)
    if uneven:
        a_old = _a_old("uneven", a_old + np.float32(0.01), np.random.default_rng(N))
    return x, y, z, m, a_old


def _params(**kw):
    import paper_1811_02761_amd as nb
    return nb.Params(**kw)


@pytest.mark.parametrize("comp", [0, 1])
@pytest.mark.parametrize("uneven", [False, True])
def test_leaf_in_slices_matches_oracle(nb, torch, orc, uneven, comp):
    _say("over-full leaf, uneven a_old", uneven, "compensated", comp)
    x, y, z, m, a_old = _input(orc, uneven)
    params = nb.Params(compensated=comp)
    ctx, acc = _run(nb, torch, x, y, z, m, params, a_old=a_old)
    ref = _ref(orc, x, y, z, m, params, a_old)
    assert ref.gentries.max() > 10000
    _, et = _compare_walk(nb, ctx, ref, acc, np.stack([x, y, z], 1), m, 2.0 ** -7)
    # (the forces of coincident particles cancel: e has no scale)
    if comp:
        _assert_rule(et, et)
    else:
        # 6000 equal terms round alike: a running sum of k terms is off by up to k
        # roundings of 2^-24 of the terms' sum, and a list has four
        assert et.max() <= (ref.gentries.max() / 4 + 16) * 2.0 ** -24


@pytest.mark.parametrize("comp", [0, 1])
@pytest.mark.parametrize("uneven", [False, True])
def test_leaf_in_slices_does_not_depend_on_the_walk(nb, torch, orc, uneven, comp):
    x, y, z, m, a_old = _input(orc, uneven)
    outs = []
    for fc, split, waves in ((0, 0, 32), (64, 2, 4), (512, 1, 12), (0, 1, 1)):
        outs.append(_run(nb, torch, x, y, z, m,
                         nb.Params(frontier_cap=fc, walk_split=split, waves_per_cu=waves,
                                   compensated=comp), a_old=a_old)[1])
    out = tuple(torch.empty(N, dtype=torch.float32, device="cuda") for _ in range(3))
    nb.tree_forces_noalloc(nb.Params(compensated=comp),
                           *(_dev(torch, a) for a in (x, y, z, m)),
                           tuple(_dev(torch, a_old[:, k]) for k in range(3)), out)
    outs.append(np.stack([_np(t) for t in out], 1))
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])
