"""The list of the first round after blocks are solved apart: columns that are
pivots as they are, in complexes of two to five dimensions (some blocks solved,
some not), with matrices ending around the tiles of 1024 columns."""
import numpy as np
import pytest

from tests import brute
from tests.test_gpu_graph import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_dim", [2, 3, 4, 5])
@pytest.mark.parametrize("m", [0, 1023, 1024, 1025, 2049])
def test_first_list(gpu, max_dim, m):
    rng = np.random.default_rng(100 * max_dim + m)
    for _ in range(6):
        cp, rows, dim, _, _ = brute.random_filtration(rng, n_vertices=int(rng.integers(max_dim + 1, 12)),
                                                      n_facets=int(rng.integers(3, 14)), max_dim=max_dim)
        n = max(m - len(dim), 0)  # vertices in front
        cols = [[] for _ in range(n)] + [[int(r) + n for r in rows[cp[j]:cp[j + 1]]] for j in range(len(dim))]
        _check(cols, [0] * n + [int(x) for x in dim], gpu)
