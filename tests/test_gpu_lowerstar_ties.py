"""Lower-star filtrations whose vertices share values, by how many do (up to
eight are placed by counting, more by sorting all simplices), scattered and
side by side, in volumes and in sheets and lines one or two vertices thin."""
import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import api
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


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 2), (1, 1, 40), (1, 2, 2), (1, 9, 13), (9, 1, 13), (2, 2, 2), (2, 9, 7), (11, 10, 9)])
def test_faces_of_the_top_simplices(gpu, shape):
    """The second cofaces that the builder gives, in one, two and three
    dimensions: the same pairs as from the matrix alone, and the oracle's."""
    n = int(np.prod(shape))
    rng = np.random.default_rng(n)
    for order in (rng.permutation(n), rng.permutation(n) // 3, np.arange(n)):
        g = torch.as_tensor(order.reshape(shape).astype(np.float32), device=gpu)
        f = api.build_lowerstar(g)
        ref = oracle.build_lowerstar(g.cpu().numpy())
        want = oracle.reduce_twist(ref.col_ptr, ref.rows, ref.dim)
        a = api.reduce_filtration(f)
        t = f.to_torch()
        b = api.reduce(t["col_ptr"], t["rows"], t["dim"])
        for r in (a, b):
            assert np.array_equal(r.low_star.cpu().numpy(), want)
            assert np.array_equal(r.essential.cpu().numpy(), oracle.essential(want))
        assert (a.rounds, a.additions) == (b.rounds, b.additions)
