"""The sweep kernel's larger sizes (columns that overfill its list in LDS, in
matrices of more than 2^23 columns) against the oracle, at list lengths of each
size and beyond the last, and the capped walks of a round that hands over more
columns than the sweeps take."""
import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import api
from tests.test_gpu_solve import _check, _counts, _csc, _reduce, sweeps_always  # noqa: F401

pytestmark = pytest.mark.gpu


def _touches(base, pivots, entries, seed):
    """`pivots` pivots of `entries` entries each among `base` rows, and three
    columns whose chains add them all; empty columns up to 2^23 + 1."""
    rng = np.random.default_rng(seed)
    tail = [sorted(rng.choice(base, entries, replace=False).tolist()) + [base + a] for a in range(pivots)]
    seen = np.unique(np.concatenate([np.asarray(t[:-1]) for t in tail])).size + pivots
    for x in (3, 7, 11):
        tail.append([x] + [base + a for a in range(pivots)])
    cols = [[] for _ in range((1 << 23) + 1)]
    return *_csc(cols + tail), seen


@pytest.mark.parametrize("base,pivots,entries,least,most", [
    (9000, 20, 1500, 6144, 12288),       # the second size
    (12200, 40, 2500, 12200, 49152),     # an edge of the second
    (45000, 60, 2800, 12288, 49152),     # the third
    (90000, 80, 2500, 49152, 1 << 30),   # none: the serial walk
])
def test_lists_of_each_size(gpu, capfd, sweeps_always, base, pivots, entries, least, most):  # noqa: F811
    cp, rows, seen = _touches(base, pivots, entries, base)
    assert least < seen <= most
    _check(_reduce(cp, rows, gpu), oracle.reduce_standard(cp, rows))
    err = capfd.readouterr().err
    assert sum(_counts(err, "to k_chain")) >= 3, err[-2000:]
    steps = sum(sum(_counts(err, name)) for name in ("chain steps short", " long", " global"))
    assert (steps > 0) == (seen > 49152), err[-2000:]


def test_capped_walks_equal_whole_ones(gpu, monkeypatch, capfd):
    monkeypatch.setenv("PMS_TRACE", "1")
    rng = np.random.default_rng(5)
    f = api.build_lowerstar(torch.as_tensor(rng.permutation(48**3).reshape(48, 48, 48).astype(np.float32), device=gpu))
    a = api.reduce_filtration(f)
    err = capfd.readouterr().err
    assert max(_counts(err, "handed to waves")) > 1024, err[-2000:]
    b = api.reduce_filtration(f, variant=1)
    for name in ("low_star", "pair_birth", "pair_death", "essential"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
