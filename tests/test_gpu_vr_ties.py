"""Many clouds with edges of equal value in groups of every size the counting
handles, wherever they fall among the steps of 64 edges of a column's pass."""
import numpy as np
import pytest

from tests.test_gpu_vr_edges import _same_as_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,n,clouds", [(60, 64, 40), (30, 48, 40), (150, 90, 12), (16, 40, 20)])
def test_groups_across_steps(gpu, side, n, clouds):
    rng = np.random.default_rng(n)
    x = [rng.integers(0, side, (n - int(rng.integers(0, 3)), 2)).astype(np.int32) for _ in range(clouds)]
    _same_as_oracle(x, [-1] * clouds, 2, gpu)


@pytest.mark.parametrize("side,n,clouds", [(90, 24, 12), (300, 34, 8)])
def test_groups_in_dimension_three(gpu, side, n, clouds):
    rng = np.random.default_rng(n)
    x = [rng.integers(0, side, (n, 3)).astype(np.int32) for _ in range(clouds)]
    _same_as_oracle(x, [-1] * clouds, 3, gpu)
