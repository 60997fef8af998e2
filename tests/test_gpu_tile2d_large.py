"""The 2-D tiles of grids from pitch 2048 (64 by 20 points, whole and ragged) in
each format, also next to a coarse level of another one: the cycle equals the
stage kernels bit for bit."""
import pytest

from tests import test_gpu_tile2d as tiles

pytestmark = pytest.mark.gpu
_gpu = tiles._gpu


@pytest.mark.parametrize("n,disc,fmt,nu1,nu2", [
    (2047, "fd", ["f64"], 2, 2), (2047, "fd", ["f32", "f16"], 1, 3), (2047, "fd", ["f16", "bf16"], 3, 1),
    (2303, "q1", ["bf16", "f64"], 2, 2), (2303, "q1", ["f64"], 3, 3)])
def test_large_tiles_equal_the_stages(n, disc, fmt, nu1, nu2):
    tiles.test_tile_cycle_equals_the_stages(n, disc, fmt, nu1, nu2)
