"""Steps on a context whose tree or workspace was dropped, or whose tree another
call replaced, against a context that never had the old one: the same bits."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_batch import _np, _say, _state_arrays, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu

N, DT = 3000, 2.0 ** -7


def _state(nb, interval, seed=21, **kw):
    p = I.plummer(N, seed)
    return nb.State.from_numpy(p.pos, p.vel, p.mass, dt=DT, rebuild_interval=interval, **kw)


def _copy(nb, st):
    """The same state in arrays of its own."""
    names = ("x", "y", "z", "vx", "vy", "vz", "m", "ax", "ay", "az")
    return nb.State(*(getattr(st, k).clone() for k in names), t=st.t, dt=st.dt,
                    have_acc=st.have_acc, rebuild_interval=st.rebuild_interval,
                    integrator=st.integrator)


def _same(a, b):
    for u, v in zip(_state_arrays(a), _state_arrays(b)):
        np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("integrator", [0, 1])
def test_steps_after_other_systems(nb, torch, integrator):
    _say("eager steps after set_systems, integrator", integrator)
    ctx = nb.Context(nb.Params(), n_max=N)
    ctx.set_systems([0, 1000, N])
    a = _state(nb, 100, integrator=integrator)
    ctx.step(a, 2)
    b = _copy(nb, a)
    ctx.set_systems([0, 500, 1700, N])
    ctx.step(a, 2)
    fresh = nb.Context(nb.Params(), n_max=N)
    fresh.set_systems([0, 500, 1700, N])
    fresh.step(b, 2)
    _same(a, b)


def _rebind(nb, torch, ctx, n_max):
    import ctypes as C
    size, cp = C.c_size_t(), ctx.params.c()
    assert nb.lib().nbody_workspace_query(C.byref(cp), n_max, C.byref(size)) == 0
    ws = torch.empty(size.value + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    ctx.sync()
    assert nb.lib().nbody_bind_workspace(ctx._h, C.c_void_p(base), size.value, n_max) == 0
    ctx.ws = ws


@pytest.mark.parametrize("interval", [2, 100])
@pytest.mark.parametrize("change", ["none", "systems", "block", "build", "workspace", "order"])
def test_graph_steps_after_other_calls(nb, torch, change, interval):
    _say("graph steps after", change, "rebuild interval", interval)
    ends = []
    for graph in (True, False):
        ctx = nb.Context(nb.Params(), n_max=N)
        st = _state(nb, interval)
        step = ctx.step_graph if graph else ctx.step
        for rep in range(3):
            step(st, 3)
            if change == "systems":
                ctx.set_systems([0, 500 + 100 * rep, N])
            elif change == "block":  # (in key order: the tree's permutation moves)
                p = I.plummer(N, 30 + rep)
                ctx.set_step_layout(1)
                ctx.step(nb.State.from_numpy(p.pos, p.vel, p.mass, dt=2.0 ** -3,
                                             rebuild_interval=2, block_steps=True), 3)
            elif change == "build":
                ctx.build_tree(*(t.float() for t in (st.x, st.y, st.z)), st.m)
            elif change == "workspace":
                _rebind(nb, torch, ctx, N + 1000 * (rep + 1))
            elif change == "order":
                ctx.set_order(rep % 2)
            step(st, 2)
            ctx.step(st, 1)  # (an eager refit of the tree the replays left)
        ctx.sync()
        ends.append((st, ctx.export(nb.X.PERM).cpu().numpy(), ctx.stats()))
    _same(ends[0][0], ends[1][0])
    np.testing.assert_array_equal(ends[0][1], ends[1][1])
    for k in ("steps", "rebuilds", "ncell", "list_entries", "queued"):
        assert ends[0][2][k] == ends[1][2][k], k


def test_systems_stay_with_another_workspace(nb, torch):
    off = [0, 700, 1900, N]
    ctx, want = nb.Context(nb.Params(order=2), n_max=N), nb.Context(nb.Params(), n_max=N)
    ctx.set_cost_model(8, torch.ones(nb.mlp_nparams(8), device="cuda"))
    ctx.set_systems(off)
    want.set_systems(off)
    a, b = _state(nb, 2), _state(nb, 2)
    ctx.step(a, 2)
    old = ctx.ws
    _rebind(nb, torch, ctx, N + 5000)
    old.fill_(255)  # (nothing of the old memory is used again)
    ctx.step(a, 2)
    want.step(b, 4)
    ctx.sync()
    assert ctx.stats()["queued"] == ctx.stats()["ngroup"]
    # (the tree was dropped after the second step, so both rebuild before the third)
    _same(a, b)
