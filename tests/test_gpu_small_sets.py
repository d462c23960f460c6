"""Tree builds at the edges of the paths chosen by the particle count, against
the CPU oracle: calcNode's ranges (one, four or sixteen chunks of 64 particles
per wavefront)."""
import pytest

import nbody_inputs as I
from test_gpu_parity import _compare_tree, _ref, _run, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [255, 256, 257, 1000, 4097, 32767, 32768, 65537])
def test_tree_at_path_edges(nb, torch, orc, n):
    g = I.galaxy(n, 17)
    x, y, z, _, _, _, m = g.f32()
    params = nb.Params()
    ctx, _ = _run(nb, torch, x, y, z, m, params)
    _compare_tree(nb, ctx, _ref(orc, x, y, z, m, params), torch)
