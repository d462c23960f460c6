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
