"""Inputs at the edge of what scratch, views and tables are sized for."""
import numpy as np
import pytest

from paper_1708_04710_amd import synth
from tests.test_gpu_build import _compare_lowerstar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 64, 64), (1, 300, 300), (301, 1, 299), (1, 500, 500), (1, 1, 4099), (1, 1, 100_000)])
@pytest.mark.parametrize("levels", [0, 50])
def test_flat_grids(gpu, shape, levels):
    """Images and lines: few simplices a vertex, so more tiles of vertices than
    of simplices (1 024 bytes of tile sums against 960 of the other for 64 x 64)."""
    g = synth.random_grid(71, shape)
    if levels:
        g = np.floor(g * levels).astype(np.float32)
    _compare_lowerstar(g, gpu)
