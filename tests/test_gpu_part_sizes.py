"""Heavy groups at both sides of the tree size where their parts change size
(256 and 512 particles), against the CPU oracle under the rules of
test_gpu_heavy.py."""
import pytest

from test_gpu_heavy import test_heavy_groups_match_oracle as check
from test_gpu_parity import nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32768, 32769])
def test_parts_on_both_sides(nb, torch, orc, n):
    check(nb, torch, orc, "plummer", n, 2.0 ** -9, True, 0)
