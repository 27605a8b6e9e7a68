"""The fp32 grouped GEMMs at the edges of their tiles: the 64-row tiles (taken from an
average of 48 rows per expert on), with experts of 1 row, either side of the 32-row
blocks and of the 64-row tile, and of several tiles; the 32-row tiles with fewer rows.
Weight gradients contract over the rows in stages of 32 and groups of 8: counts off both.
D and H are one and several 64-wide column tiles.  Forward, backward and the SGD update
against the oracle's expert block at the fp32 tolerance."""
import pytest

from test_gpu_expert_rows import check_expert_calls

pytestmark = pytest.mark.gpu

CASES = {
    "f32_64_rows": dict(d=2, M=3, D=192, H=320, seed=74, dtype="f32", counts=[64, 1, 63, 65, 0, 129, 200, 96, 33]),
    "f32_64_rows_narrow": dict(d=1, M=4, D=64, H=64, seed=75, dtype="f32", counts=[127, 0, 128, 7]),
    "f32_32_rows": dict(d=2, M=4, D=128, H=192, seed=76, dtype="f32",
                        counts=[1, 0, 2, 7, 8, 9, 15, 31, 32, 33, 40, 41, 3, 0, 100, 5]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_f32_expert_calls_on_tile_edges(name):
    check_expert_calls(name, CASES[name])
