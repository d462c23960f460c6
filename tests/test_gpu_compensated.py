"""The compensated sum is compensated in every form of the walk. Half of the
particles lie next to one point, so a list holds thousands of like terms, whose
roundings in a plain sum go the same way: with plain sums accelerations are further
from the direct FP64 sum than the roundings of a term allow, in the same lists; with
compensated sums none is. delta_acc = 0: every particle is an entry, and the groups'
lists are split or not. With an a_old that is tiny and differs from particle to
particle every particle is an entry too, and every group is walked in parts, the
over-full leaf in slices (with one wavefront per CU there is no room for most parts:
their sums are made one after the other)."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import _dev, _np, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu
# each term: at most about 8 roundings of 2^-24; the result adds one
BOUND = 9 * 2.0 ** -24


@pytest.mark.parametrize("n,parts,split,waves", [
    (3001, False, 1, 32), (3001, False, 2, 32), (60001, False, 0, 32), (60001, False, 1, 32),
    (40001, True, 0, 32), (40001, True, 0, 1)])
def test_sums_stay_compensated(nb, torch, n, parts, split, waves):
    _say("compensated", n, "parts", parts, "split", split, "wavefronts per CU", waves)
    x, y, z, _, _, _, m = I.plummer(n, 61).f32()
    k, rng = np.arange(0, n, 2), np.random.default_rng(n)
    for a, at in zip((x, y, z), (0.71, -0.43, 0.57)):
        # (not quite one point: a leaf of no size at all is a single entry)
        a[k] = at + rng.integers(-4, 5, len(k)) * 2.0 ** -24
    X, Y, Z, M = (_dev(torch, a) for a in (x, y, z, m))
    tiny = tuple(_dev(torch, (10.0 ** rng.uniform(-18, -16, n)).astype(np.float32))
                 for _ in range(3))
    off = {}
    for comp in (0, 1):
        ctx = nb.Context(nb.Params(compensated=comp, walk_split=split, waves_per_cu=waves,
                                   delta_acc=2.0 ** -9 if parts else 0.0), n_max=n)
        ctx.build_tree(X, Y, Z, M)
        acc, _ = ctx.calc_acc_pot(tiny if parts else ctx.calc_acc(None))
        want, scale, _ = ctx.direct64(X, Y, Z, M, torch.arange(n, device="cuda"))
        err = (torch.stack(list(acc), 1).double() - want).abs().amax(1) / scale
        off[comp] = _np(err)
    plain = np.percentile(np.delete(off[0], k), 99)  # (the point's own have no such terms)
    _say("  plain sums off by %.1f, compensated at most %.2f bounds"
         % (plain / BOUND, off[1].max() / BOUND))
    assert plain > BOUND
    assert (off[1] <= BOUND).all()
