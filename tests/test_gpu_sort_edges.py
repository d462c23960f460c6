"""The sort at the edges of its tiles and of the ranges that choose them (places
counted in tiles of 1024 or 4096, tiles sorted by digits), against a stable
sort of the same keys in numpy."""
import numpy as np
import pytest

from test_gpu_parity import nb, torch  # noqa: F401
from test_gpu_small_sets import test_sort_is_stable as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [255, 256, 257, 1023, 1024, 1025, 4161, 32767, 32768, 32769,
                               33793, 131072, 131073])
@pytest.mark.parametrize("grid", [0, 5])
def test_sort_at_tile_edges(nb, torch, n, grid):
    check(nb, torch, n, grid)
