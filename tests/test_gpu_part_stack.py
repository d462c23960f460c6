"""A part of a heavy group that outgrows its stack: k_heavy_walk hands the group on and
k_heavy_end walks it again, with the sums of parts that fit. The input is made for it:
one group's box spans the whole root cube, its front stops at 512 cells of 2100
particles (4096 more would not fit), and one of these cells holds a chain of nested
corners, each with 64 grandchildren of 8 children, so that a depth-first stack of the
cell's subtree passes 4096 cells. With frontier_cap = 16384 the parts' stacks hold all.

The same for heavy groups inside replayed steps: graph and eager steps end alike."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import _dev, _np, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _corner_chain():
    """Positions in the unit cell: the centres of the children of all grandchildren of
    C_0 = the cell, C_1 = its last octant, ..., C_10."""
    g = np.stack(np.meshgrid(*[np.arange(8)] * 3, indexing="ij"), -1).reshape(-1, 3)
    out = []
    for lv in range(11):
        size = 0.5 ** lv
        p = (1.0 - size) + (g + 0.5) / 8 * size
        out.append(p if lv == 10 else p[(p < 1.0 - size / 2).any(1)])
    return np.concatenate(out)


def _input():
    rng = np.random.default_rng(9)
    cells = np.stack(np.meshgrid(*[np.arange(8, 16)] * 3, indexing="ij"), -1).reshape(-1, 3) / 16
    pos = (cells[:-1, None, :] + rng.uniform(0.002, 0.998, (511, 2100, 3)) / 16).reshape(-1, 3)
    pos = np.concatenate([pos, cells[-1] + _corner_chain() / 16])
    far = []  # eight particles in each of the other octants, the cube's corners among them
    for o in range(7):
        at = np.array([o >> 2 & 1, o >> 1 & 1, o & 1]) * 0.5
        far.append(at + rng.uniform(0.05, 0.45, (8, 3)))
        far[-1][0] = np.where(at > 0, 0.999999, 1e-6)
    pos = np.concatenate([pos] + far)
    n = len(pos)
    a = np.full(n, 1e6, np.float32)  # (everyone else's lists are short)
    a[-56:] = 10.0 ** rng.uniform(-6, -4, 56)
    return pos.astype(np.float32), np.full(n, 1.0 / n, np.float32), a


def _deepest_stack(first, nchild, cell):
    """Most cells on a walk's stack that starts with `cell` and opens every cell."""
    stack, most = [cell], 1
    while stack:
        top, stack = stack[-64:], stack[:-64]
        for c in top:
            stack += range(first[c], first[c] + nchild[c])
        most = max(most, len(stack))
    return most


@pytest.mark.parametrize("comp", [0, 1])
def test_part_that_outgrows_its_stack(nb, torch, comp):
    pos, m, a = _input()
    n = len(m)
    _say("part stack", n, "compensated", comp)
    X, Y, Z, M, A = (_dev(torch, np.ascontiguousarray(v)) for v in (*pos.T, m, a))
    zero = torch.zeros_like(A)
    res = []
    for fc in (0, 16384):
        ctx = nb.Context(nb.Params(leaf_max=1, compensated=comp, checks=1, frontier_cap=fc),
                         n_max=n)
        ctx.build_tree(X, Y, Z, M)
        acc = ctx.calc_acc((A, zero, zero))
        res.append([_np(t) for t in acc] + [_np(ctx.export(k)) for k in (nb.X.GENTRIES,
                                                                        nb.X.GHASH)])
    lev, cnt, fch, nch = (_np(ctx.export(k)) for k in (nb.X.LEVEL, nb.X.PCOUNT, nb.X.FCHILD,
                                                       nb.X.NCHILD))
    cell = np.flatnonzero((lev == 4) & (cnt == len(_corner_chain())))
    assert len(cell) == 1 and (cnt[lev == 4] > 2048).sum() == 512
    assert _deepest_stack(fch, nch, int(cell[0])) > 4096
    assert res[0][3].max() > n // 2  # (the one group that meets every particle)
    for u, v in zip(*res):
        np.testing.assert_array_equal(u, v)
    t = torch.arange(n - 56, n, device="cuda")
    want, scale, _ = ctx.direct64(X, Y, Z, M, t)
    err = np.abs(np.stack(res[0][:3], 1)[-56:] - _np(want)).max(1) / _np(scale)
    assert err.max() <= 1e-3  # (every term a particle or a small accepted cell)


def test_heavy_groups_in_replayed_steps(nb, torch):
    n = 30011
    p = I.plummer(n, 31)
    ends = []
    for graph in (False, True):
        ctx = nb.Context(nb.Params(), n_max=n)
        st = nb.State.from_numpy(p.pos, p.vel, p.mass, dt=2.0 ** -8, rebuild_interval=2)
        for _ in range(4):
            (ctx.step_graph if graph else ctx.step)(st, 2)
            _ = (torch.ones(1000, device="cuda") * 2).sum().item()  # (eager work in between)
        ctx.sync()
        assert int(ctx.export(nb.X.GENTRIES).max()) > 4096
        ends.append([_np(t) for t in (st.x, st.y, st.z, st.vx, st.vy, st.vz, st.ax, st.ay, st.az)])
    for u, v in zip(*ends):
        np.testing.assert_array_equal(u, v)
