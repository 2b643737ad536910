"""The first addition of a round's colliding columns by the whole workgroup
(long merges) against the oracle: lengths at the edges of its pieces of 2048
entries and of the lane merges, entries that cancel across pieces and threads,
and more long columns in a tile than it takes."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_solve import _check, _csc, _reduce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", [1, 3, 40])
@pytest.mark.parametrize("n", [32, 33, 300, 1023, 1024, 1025, 2100, 5000])
def test_long_first_additions(gpu, n, groups):
    rng = np.random.default_rng(1000 * groups + n)
    base = n + n // 2 + 8
    cols = [[] for _ in range(base + groups)]
    for g in range(groups):  # columns of one low: half their entries common, runs of them
        common = np.arange(int(rng.integers(0, n // 4 + 1)), n // 2)
        for _ in range(3):
            own = rng.choice(np.arange(n // 2, base), n - 1 - common.size, replace=False)
            cols.append(sorted({*common.tolist(), *own.tolist()}) + [base + g])
    # pivots of some rows, so that rows are known negative: dropped by compression
    cols += [[int(r)] for r in rng.choice(base, base // 8, replace=False)]
    cp, rows = _csc(cols)
    want = oracle.reduce_standard(cp, rows)
    for kw in (dict(), dict(variant=1), dict(compression=False)):
        _check(_reduce(cp, rows, gpu, **kw), want)
