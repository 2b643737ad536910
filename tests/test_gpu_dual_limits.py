"""Blocks reduced from their rows whose lists are full (the rounds take over), whose
bitmap moves on, and whose counters are reset between rounds: the results are
those of the oracle whatever the limits are."""
import contextlib

import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import _binding as B
from paper_1708_04710_amd import api

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def _limits(gpu, sum=0, arena=0, beyond=0, bits=0, rounds=0):
    ctx, lib = api._ctx(gpu), B.load()
    B.check(ctx, lib.pms_set_dual_limits(ctx, sum, arena, beyond, bits, rounds))
    try:
        yield
    finally:
        B.check(ctx, lib.pms_set_dual_limits(ctx, 0, 0, 0, 0, 0))


def _clouds(seed, n, count, kind):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(count):
        p = rng.normal(size=(n, 3))
        if kind == "circle":
            a = rng.uniform(0, 2 * np.pi, n)
            p = np.stack([np.cos(a), np.sin(a), np.zeros(n)], 1)
        elif kind == "sphere":
            p /= np.linalg.norm(p, axis=1, keepdims=True)
        out.append(np.rint(p * 5000 + rng.normal(0, 120, p.shape)).astype(np.int32))
    return out


def _want(clouds, maxdim):
    refs = [oracle.build_vr_i32(c, maxdim=maxdim) for c in clouds]
    low, off = [], [0]
    for r in refs:
        w = oracle.reduce_twist(r.col_ptr, r.rows, r.dim)
        low.append(np.where(w >= 0, w + off[-1], -1))
        off.append(off[-1] + r.m)
    return np.concatenate(low), off


def _check(res, want, off=None):
    assert np.array_equal(res.low_star.cpu().numpy(), want)
    b, d = oracle.pairs(want)
    assert np.array_equal(res.pair_birth.cpu().numpy(), b) and np.array_equal(res.pair_death.cpu().numpy(), d)
    assert np.array_equal(res.essential.cpu().numpy(), oracle.essential(want))
    if off is not None:
        assert np.array_equal(res.inst_pair_off.cpu().numpy(), np.searchsorted(d, off))
        assert np.array_equal(res.pair_inst.cpu().numpy(), np.searchsorted(off, d, side="right") - 1)


# limits, and whether the blocks still fit in them (None: some columns may, or all)
LIMITS = [(dict(), True), (dict(rounds=2), True), (dict(rounds=4), True), (dict(arena=1), False), (dict(arena=150), None)]


@pytest.mark.parametrize("limits,fits", LIMITS)
def test_edges_over_triangles(gpu, limits, fits):
    clouds = _clouds(5, 60, 6, "circle") + _clouds(6, 48, 4, "ball")
    want, off = _want(clouds, 2)
    f, dev_off = api.build_vr([torch.as_tensor(c, device=gpu) for c in clouds])
    plain = api.reduce_batched(f, dev_off)
    with _limits(gpu, **limits):
        res = api.reduce_batched(f, dev_off)
    _check(res, want, off)
    assert fits is None or (res.additions == plain.additions) == fits
    assert plain.rounds > 3  # (block 0 is one; more than two for the counters to be reset)


@pytest.mark.parametrize("limits,fits", LIMITS + [(dict(sum=1), False), (dict(sum=20), None), (dict(bits=1024), True),
                                                 (dict(bits=5000, rounds=2), True), (dict(bits=1024, beyond=3), False)])
@pytest.mark.parametrize("count", [1, 3])
def test_triangles_over_tetrahedra(gpu, limits, fits, count):
    clouds = _clouds(7, 34, count, "sphere")
    want, off = _want(clouds, 3)
    f, dev_off = api.build_vr([torch.as_tensor(c, device=gpu) for c in clouds], None, 3)
    plain = api.reduce_batched(f, dev_off)
    with _limits(gpu, **limits):
        res = api.reduce_batched(f, dev_off)
    _check(res, want, off)
    assert fits is None or (res.additions == plain.additions) == fits


@pytest.mark.parametrize("limits,fits", LIMITS + [(dict(sum=1), False), (dict(sum=9), None), (dict(bits=1024), False)])
@pytest.mark.parametrize("maxdim,n", [(2, 60), (3, 30)])
def test_matrix(gpu, limits, fits, maxdim, n):
    cloud = _clouds(8, n, 1, "circle" if maxdim == 2 else "sphere")
    want, _ = _want(cloud, maxdim)
    f, _ = api.build_vr(torch.as_tensor(cloud[0], device=gpu), None, maxdim)
    t = f.to_torch()
    args = t["col_ptr"], t["rows"], t["dim"]
    plain = api.reduce(*args)
    for noalloc in (False, True):
        with _limits(gpu, **limits):
            res = api.reduce(*args, noalloc=noalloc)
        _check(res, want)
        assert fits is None or (res.additions == plain.additions) == fits


def test_limits_out_of_range_are_refused(gpu):
    for bad in (dict(sum=-1), dict(bits=1000), dict(bits=1 << 21), dict(rounds=3), dict(rounds=258)):
        with pytest.raises(B.PmsError) as e, _limits(gpu, **bad):
            pass
        assert e.value.status == B.PMS_ERR_INVALID_ARG


@pytest.mark.parametrize("maxdim,n", [(2, 60), (3, 30)])
def test_bytes_of_the_additions(gpu, maxdim, n):
    """Of these clouds nothing is left to the rounds, so every entry read is one
    toggled in place (8 bytes), as a filtration and as a matrix."""
    cloud = _clouds(8, n, 1, "circle" if maxdim == 2 else "sphere")[0]
    f, _ = api.build_vr(torch.as_tensor(cloud, device=gpu), None, maxdim)
    t = f.to_torch()
    for res in (api.reduce_filtration(f), api.reduce(t["col_ptr"], t["rows"], t["dim"])):
        assert res.xor_entries > 0 and res.addition_bytes == 8 * res.xor_entries
