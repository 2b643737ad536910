"""Vietoris-Rips filtrations built by edge order, and their reduction from the
faces' side, against the oracle: word and wavefront edges of the masks, no
and few points, coincident points, tie groups below and above the counted
size, both edge sorts, every dimension."""
import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import api, synth
from tests.test_gpu_build import _compare_vr

pytestmark = pytest.mark.gpu


def _same_as_oracle(clouds, thrs, maxdim, gpu):
    f, off, refs = _compare_vr(clouds, thrs, maxdim, gpu)
    want = []
    for b, ref in enumerate(refs):
        low = oracle.reduce_twist(ref.col_ptr, ref.rows, ref.dim) if ref.m else np.zeros(0, np.int32)
        want.append(np.where(low >= 0, low + off[b], -1))
    low = np.concatenate(want).astype(np.int32)
    for res in (api.reduce_batched(f, off), api.reduce_filtration(f)):
        got = res.low_star.cpu().numpy()
        bad = np.flatnonzero(got != low)
        assert bad.size == 0, f"{bad.size} columns differ, first {bad[:5]}"
        b, d = oracle.pairs(low)
        assert np.array_equal(res.pair_birth.cpu().numpy(), b) and np.array_equal(res.pair_death.cpu().numpy(), d)
        assert np.array_equal(res.essential.cpu().numpy(), oracle.essential(low))


@pytest.mark.parametrize("n", [1, 2, 3, 31, 32, 33, 63, 64, 65, 127, 129])
@pytest.mark.parametrize("f32", [False, True])
def test_sizes_around_words(gpu, n, f32):
    rng = np.random.default_rng(n)
    p = rng.normal(size=(n, 3)).astype(np.float32) if f32 else rng.integers(0, 1 << 14, (n, 3)).astype(np.int32)
    _same_as_oracle([p], [-1.0 if f32 else -1], 2, gpu)


@pytest.mark.parametrize("maxdim", [0, 1, 2, 3])
def test_uneven_batch_with_empty_clouds(gpu, maxdim):
    rng = np.random.default_rng(40 + maxdim)
    sizes = [0, 5, 1, 40, 2, 0, 33, 17]
    clouds = [rng.integers(0, 1 << 15, (n, 2)).astype(np.int32) for n in sizes]
    thrs = [-1, 1 << 28, -1, 1 << 29, 0, -1, 1 << 27, -1]
    _same_as_oracle(clouds, thrs, maxdim, gpu)


@pytest.mark.parametrize("side,n,maxdim", [(400, 70, 2), (40, 60, 2), (12, 40, 2), (3, 30, 2), (40, 24, 3), (200, 30, 3), (90, 40, 3), (1, 9, 2)])
def test_edges_of_equal_value(gpu, side, n, maxdim):
    """Coarse integer points: pairs, small groups and (side 3, 1) groups of
    hundreds of edges of one value, coincident points among them."""
    rng = np.random.default_rng(side)
    clouds = [rng.integers(0, side, (n + k, 2)).astype(np.int32) for k in range(3)]
    _same_as_oracle(clouds, [-1, side * side // 2, -1], maxdim, gpu)


@pytest.mark.parametrize("n,pct", [(200, 1.0), (300, 0.3), (505, 0.04), (420, 0.25)])
def test_both_edge_sorts(gpu, n, pct):
    """Up to 16 384 edges in one workgroup, beyond that device-wide (the full
    200 points: 19 900; 420 points at 0.25: 21 998), also mixed in one batch."""
    rng = np.random.default_rng(n)
    big = rng.integers(0, 1 << 16, (n, 2)).astype(np.int32)
    small = rng.integers(0, 1 << 16, (20, 3)).astype(np.int32)
    thr = -1 if pct == 1.0 else synth.percentile_threshold_sqd(big, pct)
    _same_as_oracle([small, big, small + 1], [-1, thr, 1 << 30], 2, gpu)


def test_dimension_three_batch(gpu):
    x = synth.circle_batch(seed=9, clouds=3, n=34)
    _same_as_oracle(list(x), [-1.0, 1.5, -1.0], 3, gpu)
    pts, thr = synth.vr_torus(n=150)
    _same_as_oracle([pts], [thr], 3, gpu)


def test_a_workspace_reused_by_other_builders(gpu):
    """One Filtration rebuilt by the cloud builder in dimension 3, 2, with
    many ties, and by the volume builder, reduced each time."""
    rng = np.random.default_rng(3)
    f = api.Filtration(torch.device("cuda", torch.cuda.current_device()))
    a = rng.integers(0, 1 << 14, (40, 3)).astype(np.int32)
    t = rng.integers(0, 3, (40, 2)).astype(np.int32)
    g = synth.random_grid(5, (6, 7, 8))
    for kind in (3, 2, "ties", 2, "grid", 3, "grid"):
        if kind == "grid":
            api.build_lowerstar(torch.as_tensor(g, device=gpu), out=f)
            ref = oracle.build_lowerstar(g)
        else:
            p, d = (t, 2) if kind == "ties" else (a, kind)
            api.build_vr([torch.as_tensor(p, device=gpu)], [-1], d, out=f)
            ref = oracle.build_vr_i32(p, -1, d)
        res = api.reduce_filtration(f)
        assert np.array_equal(res.low_star.cpu().numpy(), oracle.reduce_twist(ref.col_ptr, ref.rows, ref.dim))
