"""Trees on both sides of the size from which the internal cells' block counts
are scanned by a launch of their own (4096 blocks of 256 cells of the most that
n particles can make), against the CPU oracle."""
import pytest

import nbody_inputs as I
from test_gpu_parity import _compare_tree, _ref, _run, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [469098, 469100])
def test_tree_where_the_scan_changes(nb, torch, orc, n):
    x, y, z, _, _, _, m = I.galaxy(n, 23).f32()
    params = nb.Params()
    ctx, _ = _run(nb, torch, x, y, z, m, params)
    _compare_tree(nb, ctx, _ref(orc, x, y, z, m, params), torch)
