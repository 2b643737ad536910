"""Rounds whose ends run in one workgroup, against the oracle and against the
rounds of a captured graph (one kernel per step): active columns at the edges
of a thread's share, of the wavefronts and of the limits, and results that do
not fit the caller's arrays."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import _binding as B
from paper_1708_04710_amd import api
from tests.test_gpu_solve import _check, _csc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
def test_round_edges(gpu, n):
    rng = np.random.default_rng(n)
    base = max(3, n // 2)
    cols = [[] for _ in range(base)]
    for _ in range(n):
        cols.append(sorted(rng.choice(base, size=int(rng.integers(1, min(base, 6) + 1)), replace=False).tolist()))
    cp, rows = _csc(cols)
    want = oracle.reduce_standard(cp, rows)
    args = [torch.as_tensor(x, device=gpu) for x in (cp, rows)]
    a = api.reduce(*args, None, validate=False)
    b = api.reduce(*args, None, validate=False, graph_rounds=2)
    _check(a, want)
    _check(b, want)
    assert (a.rounds, a.additions) == (b.rounds, b.additions)


def test_nothing_written_when_it_does_not_fit(gpu):
    cols = [[], [], [], [0, 1], [1, 2], [0, 2]]
    cp, rows = (torch.as_tensor(x, device=gpu) for x in _csc(cols))
    ctx, lib = api._ctx(torch.device(gpu)), B.load()
    out = [torch.full((4,), -7, dtype=torch.int32, device=gpu) for _ in range(3)]
    low = torch.empty(6, dtype=torch.int32, device=gpu)
    bnd = B.PmsBoundary(m=6, col_ptr=cp.data_ptr(), rows=rows.data_ptr())
    opt = lib.pms_default_options()
    for caps in ((1, 4), (4, 1)):
        res = B.PmsResult(low_star=low.data_ptr(), pair_birth=out[0].data_ptr(), pair_death=out[1].data_ptr(),
                          cap_pairs=caps[0], essential=out[2].data_ptr(), cap_essential=caps[1])
        assert lib.pms_reduce(ctx, ctypes.byref(bnd), ctypes.byref(opt), ctypes.byref(res)) == B.PMS_ERR_CAPACITY
        assert (res.n_pairs, res.n_essential) == (2, 2)
        assert all(bool((o == -7).all()) for o in out)
