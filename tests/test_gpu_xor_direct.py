"""Columns queued straight for the sweep and wavefront kernels, against the
oracle and against the rounds of a captured graph (which keep the lane
passes): active columns at the edges of the limit, and columns longer than a
lane holds."""
import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import api
from tests.test_gpu_solve import _check, _csc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,base,size", [(65535, 2000, 2), (65536, 2000, 2), (65537, 2000, 2), (65, 700, 33),
                                         (300, 700, 129), (257, 1000, 600)])
@pytest.mark.parametrize("kw", [{}, dict(compression=False), dict(variant=1)])
def test_direct_queue(gpu, n, base, size, kw):
    rng = np.random.default_rng(n + size)
    cols = [[] for _ in range(base)]
    if size == 2:
        a = rng.integers(0, base - 1, n)
        b = a + 1 + rng.integers(0, base - 1 - a)
        cols += [[int(x), int(y)] for x, y in zip(a, b)]
    else:
        cols += [sorted(rng.choice(base, size=int(rng.integers(1, size + 1)), replace=False).tolist()) for _ in range(n)]
    cp, rows = _csc(cols)
    want = oracle.reduce_standard(cp, rows)
    args = [torch.as_tensor(x, device=gpu) for x in (cp, rows)]
    a = api.reduce(*args, None, validate=False, **kw)
    b = api.reduce(*args, None, validate=False, graph_rounds=2, **kw)
    _check(a, want)
    _check(b, want)
    assert (a.rounds, a.additions) == (b.rounds, b.additions)
