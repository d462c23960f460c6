"""Tree builds at the edges of the paths chosen by the particle count, against
numpy and the CPU oracle: the sort (tiles of 4096 merged four at a time up to
2^20, digit passes beyond) and calcNode's ranges (one, four or sixteen chunks
of 64 particles per wavefront)."""
import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import _compare_tree, _dev, _np, _ref, _run, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 4095, 4096, 4097, 16384, 16385, 65537, 262145,
                               (1 << 20) - 1, (1 << 20) + 1])
@pytest.mark.parametrize("grid", [0, 37])
def test_sort_is_stable(nb, torch, n, grid):
    # grid: positions on a coarse lattice, so most keys have many equals
    rng = np.random.default_rng(n + grid)
    p = rng.uniform(-1.0, 1.0, (3, n)).astype(np.float32)
    if grid:
        p = (np.floor(p * grid) / grid).astype(np.float32)
    m = np.ones(n, np.float32)
    ctx = nb.Context(nb.Params(), n_max=n)
    ctx.build_tree(*(_dev(torch, a) for a in (*p, m)))
    keys = _np(ctx.export(nb.X.KEYS))
    perm = _np(ctx.export(nb.X.PERM)).astype(np.int64)
    box = _np(ctx.export(nb.X.BOX))
    _say("sort", n, "grid", grid)
    q = np.minimum(np.floor((p.astype(np.float64) - box[:3, None]) * (2.0 ** 21 / box[3])),
                   2 ** 21 - 1).astype(np.uint64)
    k = np.zeros(n, np.uint64)
    for b in range(21):
        for a in range(3):
            k |= ((q[a] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - a)
    np.testing.assert_array_equal(perm, np.argsort(k, kind="stable"))
    np.testing.assert_array_equal(keys, k[perm])


@pytest.mark.parametrize("n", [255, 256, 257, 1000, 4097, 32767, 32768, 65537])
def test_tree_at_path_edges(nb, torch, orc, n):
    g = I.galaxy(n, 17)
    x, y, z, _, _, _, m = g.f32()
    params = nb.Params()
    ctx, _ = _run(nb, torch, x, y, z, m, params)
    _compare_tree(nb, ctx, _ref(orc, x, y, z, m, params), torch)
