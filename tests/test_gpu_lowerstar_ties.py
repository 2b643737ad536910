"""Lower-star filtrations whose vertices share values, by how many do (up to
eight are placed by counting, more by sorting all simplices), scattered and
side by side, in volumes and in sheets and lines one or two vertices thin."""
import numpy as np
import pytest

from tests.test_gpu_build import _compare_lowerstar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("same", [1, 2, 3, 7, 8, 9, 40])
@pytest.mark.parametrize("shape", [(7, 9, 11), (2, 16, 17), (1, 23, 22), (1, 1, 300), (2, 2, 2), (4, 1, 70)])
def test_shared_values(gpu, shape, same):
    n = int(np.prod(shape))
    rng = np.random.default_rng(n + same)
    for order in (np.arange(n), rng.permutation(n), np.arange(n)[::-1]):
        g = (order // same - n // (2 * same)).astype(np.float32).reshape(shape)
        _compare_lowerstar(np.ascontiguousarray(g), gpu)
