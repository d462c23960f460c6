"""Groups whose list exceeds one wavefront's limit (walked in parts: a front of
cells cut by particle counts) against the CPU oracle: every list's length and
entry hash bit for bit, forces under the tree-parity rule of
test_gpu_parity.py; the same bits from the potential walk, the allocation-free
call, small stacks (retry pass) and any split of the light groups."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import (_assert_rule, _compare_walk, _dev, _np, _ref, _run, _say,  # noqa: F401
                             nb, torch)

pytestmark = pytest.mark.gpu
LIMIT = 4096  # entries, for trees of up to 2^18 particles


def _particles(kind, n):
    if kind == "coincident":  # one level-21 leaf over the limit, and a few others
        rng = np.random.default_rng(3)
        x, y, z = (np.concatenate([np.full(n - 200, 0.25), rng.uniform(-1, 1, 200)])
                   .astype(np.float32) for _ in range(3))
        return x, y, z, np.full(n, 1.0 / n, np.float32)
    p = I.plummer(n, 31) if kind == "plummer" else I.galaxy(n, 31)
    x, y, z, _, _, _, m = p.f32()
    return x, y, z, m


# (kind, n, delta_acc, some group over the limit): the limit itself and one
# particle more, a sphere's sparse outskirts, every group heavy with fewer
# part slots than parts (the sums are then made one part after the other)
CASES = [("plummer", LIMIT, 0.0, False), ("plummer", LIMIT + 1, 0.0, True),
         ("plummer", 30011, 2.0 ** -9, True), ("galaxy", 20000, 0.0, True),
         ("coincident", 5000, 2.0 ** -9, True)]


@pytest.mark.parametrize("comp", [0, 1])
@pytest.mark.parametrize("kind,n,delta,heavy", CASES)
def test_heavy_groups_match_oracle(nb, torch, orc, kind, n, delta, heavy, comp):
    _say("heavy", kind, n, delta, "compensated", comp)
    x, y, z, m = _particles(kind, n)
    params = nb.Params(delta_acc=delta, compensated=comp)
    a_old = _ref(orc, x, y, z, m, nb.Params()).acc.astype(np.float32)
    ctx, acc = _run(nb, torch, x, y, z, m, params, a_old=a_old)
    ref = _ref(orc, x, y, z, m, params, a_old)
    assert (ref.gentries.max() > LIMIT) == heavy, ref.gentries.max()
    e, et = _compare_walk(nb, ctx, ref, acc, np.stack([x, y, z], 1), m, 2.0 ** -7)
    _say("  longest list %d, max e~ %.3g" % (ref.gentries.max(), et.max()))
    if kind == "coincident":  # (forces of coincident particles cancel: e has no scale)
        e = et
    _assert_rule(e, et)
    ao = tuple(_dev(torch, a_old[:, k]) for k in range(3))
    again, phi = ctx.calc_acc_pot(ao)
    np.testing.assert_array_equal(np.stack([_np(t) for t in again], 1), acc)
    pos = np.stack([x, y, z], 1).astype(np.float64)
    rows = np.linspace(0, n - 1, 64).astype(int)
    if delta == 0.0:  # every particle is an entry: the direct sum
        d = pos[rows][:, None, :] - pos[None, :, :]
        pij = m.astype(np.float64) / np.sqrt((d * d).sum(2) + 2.0 ** -14)
        want = -(pij.sum(1) - pij[np.arange(64), rows])
        assert np.abs(_np(phi)[rows] / want - 1).max() <= 1e-5


def test_heavy_results_do_not_depend_on_the_walk(nb, torch, orc):
    x, y, z, m = _particles("plummer", 30011)
    a_old = _ref(orc, x, y, z, m, nb.Params()).acc.astype(np.float32)
    outs = []
    for fc, split, waves in ((0, 0, 32), (64, 2, 32), (0, 1, 4), (512, 4, 12)):
        ctx, acc = _run(nb, torch, x, y, z, m,
                        nb.Params(frontier_cap=fc, walk_split=split, waves_per_cu=waves),
                        a_old=a_old)
        outs.append(acc)
    X, Y, Z, M = (_dev(torch, a) for a in (x, y, z, m))
    out = tuple(torch.empty(len(x), dtype=torch.float32, device="cuda") for _ in range(3))
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    nb.tree_forces_noalloc(nb.Params(), X, Y, Z, M, tuple(_dev(torch, a_old[:, k]) for k in range(3)),
                           out, status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    outs.append(np.stack([_np(t) for t in out], 1))
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])


def test_heavy_groups_in_a_batch_equal_separate_runs(nb, torch):
    sizes = (30011, 700, 9000)
    sets = [_particles("plummer", k) for k in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)])
    cat = [np.concatenate([s[k] for s in sets]) for k in range(4)]
    params = nb.Params(delta_acc=2.0 ** -11)
    ctx = nb.Context(params, n_max=int(off[-1]))
    ctx.set_systems(off)
    ctx.build_tree(*(_dev(torch, a) for a in cat))
    a0 = ctx.calc_acc(None)
    got = np.stack([_np(t) for t in ctx.calc_acc(a0)], 1)
    a0 = np.stack([_np(t) for t in a0], 1)
    for k, s in enumerate(sets):
        one, acc = _run(nb, torch, *s, nb.Params(delta_acc=2.0 ** -11),
                        a_old=a0[off[k]:off[k + 1]])
        np.testing.assert_array_equal(got[off[k]:off[k + 1]], acc)
        _say("system", k, "longest list", int(_np(one.export(nb.X.GENTRIES)).max()))
