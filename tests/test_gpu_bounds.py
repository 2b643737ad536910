"""Inputs at the edge of what scratch, views and tables are sized for."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import _binding as B
from paper_1708_04710_amd import api, synth
from tests import brute
from tests.test_gpu_build import _compare_lowerstar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 64, 64), (1, 300, 300), (301, 1, 299), (1, 500, 500), (1, 1, 4099), (1, 1, 100_000)])
@pytest.mark.parametrize("levels", [0, 50])
def test_flat_grids(gpu, shape, levels):
    """Images and lines: few simplices a vertex, so more tiles of vertices than
    of simplices (1 024 bytes of tile sums against 960 of the other for 64 x 64)."""
    g = synth.random_grid(71, shape)
    if levels:
        g = np.floor(g * levels).astype(np.float32)
    _compare_lowerstar(g, gpu)


def _reduce_as_given(gpu, cols, dim, **kw):
    cp = np.cumsum([0] + [len(c) for c in cols]).astype(np.int64)
    rows = np.array([r for c in cols for r in sorted(c)], np.int32)
    want = oracle.reduce_standard(cp, rows)
    args = torch.as_tensor(cp, device=gpu), torch.as_tensor(rows, device=gpu)
    for d in (torch.as_tensor(np.asarray(dim, np.int8), device=gpu), None):
        for noalloc in (False, True):
            res = api.reduce(*args, d, validate=False, noalloc=noalloc, **kw)
            assert np.array_equal(res.low_star.cpu().numpy(), want)
            b, e = oracle.pairs(want)
            assert np.array_equal(res.pair_birth.cpu().numpy(), b) and np.array_equal(res.pair_death.cpu().numpy(), e)
            assert np.array_equal(res.essential.cpu().numpy(), oracle.essential(want))
    return want


@pytest.mark.parametrize("cols,dim", [
    ([[], [0], [0]], [2, 1, 1]),             # dimensions falling: a top column named by an edge's row
    ([[], [], [0, 1]], [0, 0, 3]),           # a gap
    ([[], [], [0, 1]], [-1, -1, 0]),         # the empty simplex counted
    ([[], [0], [0], []], [1, 1, 1, 1]),      # one dimension for all
    ([[], [], [0, 1], [0, 1]], [0, 1, 1, 1]),
    ([[], [], [0, 1]], [0, -128, 127]),
])
def test_dimensions_that_are_not_those_of_facets(gpu, cols, dim):
    """Without the input check any dim is taken, and chooses slots only."""
    _reduce_as_given(gpu, cols, dim)


@pytest.mark.parametrize("seed", range(6))
def test_coboundary_matrix_with_its_simplices_dimensions(gpu, seed):
    """The anti-transpose of a boundary matrix: dim(row) = dim(column) + 1."""
    rng = np.random.default_rng(seed)
    if seed < 4:
        cp, rows, dim, _, _ = brute.random_filtration(rng, n_vertices=12, n_facets=14, max_dim=3)
    else:
        f = oracle.build_lowerstar(synth.random_grid(seed, (3, 4, 5)))
        cp, rows, dim = f.col_ptr, f.rows, f.dim
    m = len(dim)
    cols = [[] for _ in range(m)]
    for j in range(m):
        for r in rows[cp[j]:cp[j + 1]]:
            cols[m - 1 - int(r)].append(m - 1 - j)
    want = _reduce_as_given(gpu, cols, np.asarray(dim)[::-1].copy())
    assert (want >= 0).sum() == (oracle.reduce_standard(np.asarray(cp, np.int64), np.asarray(rows, np.int32)) >= 0).sum()


@pytest.mark.parametrize("what", ["as built", "left", "beta"])
def test_left_and_beta_from_the_caller(gpu, what):
    """A caller's own left and beta reach the blocks only when they are as
    defined: with others that are in range, and that the rounds do not read
    (left) or read as a bound only (beta: fewer pivots known), the pairs are the same."""
    f = api.build_lowerstar(torch.as_tensor(synth.random_grid(9, (5, 6, 7)), device=gpu))
    t = f.to_torch()
    left, beta = f.left_beta()
    want = api.reduce_filtration(f).low_star
    if what == "left":
        left = torch.full_like(left, f.m - 1)
    if what == "beta":
        beta = torch.full_like(beta, -1)
    low = torch.empty_like(want)
    bnd = B.PmsBoundary(f.m, t["col_ptr"].data_ptr(), t["rows"].data_ptr(), t["dim"].data_ptr(), left.data_ptr(),
                        beta.data_ptr())
    opt = api._options(validate=False)
    res = B.PmsResult()
    res.low_star = low.data_ptr()
    ctx = api._ctx(f.device)
    B.check(ctx, B.load().pms_reduce(ctx, ctypes.byref(bnd), ctypes.byref(opt), ctypes.byref(res)))
    assert torch.equal(low, want)


def _workspace_is_consistent(gpu, f, before):
    """After a refused build: the filtration of before, or an empty one."""
    t = f.to_torch()
    res = api.reduce_filtration(f)
    if f.m == 0:
        assert t["col_ptr"].tolist() == [0] and res.low_star.numel() == 0 and res.pair_birth.numel() == 0
        assert f.left_beta() is None
    else:
        assert f.m == before.m and np.array_equal(t["rows"].cpu().numpy(), before.rows)
        assert np.array_equal(res.low_star.cpu().numpy(), oracle.reduce_twist(before.col_ptr, before.rows, before.dim))


@pytest.mark.parametrize("first", ["grid", "cloud"])
@pytest.mark.parametrize("refused", ["grid", "cloud", "far", "arguments"])
def test_refused_build_of_a_workspace(gpu, first, refused):
    """A kept workspace built small, refused something larger, reduced, and
    built again: what it says it holds is what is reduced."""
    g = synth.random_grid(3, (4, 5, 6))
    pts = np.random.default_rng(3).integers(0, 50, (20, 3)).astype(np.int32)
    if first == "grid":
        f = api.build_lowerstar(torch.as_tensor(g, device=gpu))
        before = oracle.build_lowerstar(g)
    else:
        f, _ = api.build_vr(torch.as_tensor(pts, device=gpu))
        before = oracle.build_vr_i32(pts)
    with pytest.raises(B.PmsError) as e:
        if refused == "grid":
            bad = synth.random_grid(4, (16, 17, 18))
            bad[3, 3, 3] = np.nan
            api.build_lowerstar(torch.as_tensor(bad, device=gpu), out=f)
        elif refused == "cloud":
            bad = np.random.default_rng(5).normal(size=(90, 3)).astype(np.float32)
            bad[7, 1] = np.inf
            api.build_vr(torch.as_tensor(bad, device=gpu), out=f)
        elif refused == "far":
            api.build_vr(torch.tensor([[0], [1 << 20]], dtype=torch.int32, device=gpu), out=f)
        else:
            api.build_vr(torch.as_tensor(pts, device=gpu), maxdim=4, out=f)
    assert e.value.status == B.PMS_ERR_INVALID_ARG
    _workspace_is_consistent(gpu, f, before)
    api.build_lowerstar(torch.as_tensor(g, device=gpu), out=f)
    ref = oracle.build_lowerstar(g)
    assert np.array_equal(api.reduce_filtration(f).low_star.cpu().numpy(), oracle.reduce_twist(ref.col_ptr, ref.rows, ref.dim))
    f, off = api.build_vr([torch.as_tensor(pts, device=gpu)] * 2, out=f)
    ref = oracle.build_vr_i32(pts)
    want = oracle.reduce_twist(ref.col_ptr, ref.rows, ref.dim)
    low = api.reduce_batched(f, off).low_star.cpu().numpy()
    assert np.array_equal(low[:ref.m], want)
    assert np.array_equal(low[ref.m:], np.where(want >= 0, want + ref.m, -1))


def test_refused_first_build(gpu):
    """The same for a filtration that held nothing before."""
    f = api.Filtration(gpu)
    with pytest.raises(B.PmsError):
        api.build_lowerstar(torch.full((5, 5, 5), float("nan"), device=gpu), out=f)
    assert f.m == 0 and api.reduce_filtration(f).low_star.numel() == 0


def test_threads_with_clouds_of_other_sizes(gpu):
    """Each thread on its own stream: kernels whose dynamic LDS depends on the
    clouds are launched with 8 KB to 148 KB at once."""
    rng = np.random.default_rng(8)
    work = [(torch.as_tensor(rng.integers(0, 1 << 14, (n, 3)).astype(np.int32), device=gpu), d)
            for n, d in ((12, 2), (181, 2), (511, 2), (40, 3))]
    thr = [None, None, [1 << 22], None]

    def once(k):
        f, off = api.build_vr(work[k][0], thr[k], work[k][1])
        res = api.reduce_batched(f, off)
        return f.m, res.low_star, res.pair_birth, res.essential

    def csc(k):
        f, _ = api.build_vr(work[k][0], thr[k], work[k][1])
        t = f.to_torch()
        return f.m, api.reduce(t["col_ptr"], t["rows"], t["dim"]).low_star

    jobs = [(once, 0), (once, 1), (once, 2), (once, 3), (csc, 0), (csc, 3)]
    want = [fn(k) for fn, k in jobs]
    torch.cuda.synchronize()
    wrong = []

    def loop(i):
        fn, k = jobs[i]
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(25):
                    got = fn(k)
                    if got[0] != want[i][0] or not all(torch.equal(a, b) for a, b in zip(got[1:], want[i][1:])):
                        wrong.append((i, "differs"))
                        return
        except Exception as e:  # noqa: BLE001
            wrong.append((i, repr(e)))

    threads = [threading.Thread(target=loop, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong


@pytest.mark.parametrize("n,reverse", [(40, False), (3001, False), (30_000, False), (30_000, True)])
def test_long_strip_in_adverse_order(gpu, n, reverse):
    """Triangles (i, i+1, i+2) whose shared edges come after the boundary edges:
    they make one path through all triangles, which every boundary edge walks to
    its end.  Walked along earlier faces in one of the directions, so that the
    path is shortened (``pms_selftest`` counts the steps), along later ones in
    the other."""
    tri = np.stack([np.arange(n), np.arange(n) + 1, np.arange(n) + 2], 1)
    outer = [(0, 1), (n, n + 1)] + [(i, i + 2) for i in range(n)]
    inner = [(i + 1, i + 2) for i in range(n - 1)]
    if reverse:
        tri, inner = tri[::-1], inner[::-1]
    edges = outer + inner
    at = {e: n + 2 + k for k, e in enumerate(edges)}
    cols = [[] for _ in range(n + 2)] + [list(e) for e in edges]
    cols += [[at[(int(a), int(b))], at[(int(a), int(c))], at[(int(b), int(c))]] for a, b, c in tri]
    dim = [0] * (n + 2) + [1] * len(edges) + [2] * n
    cp = np.cumsum([0] + [len(c) for c in cols]).astype(np.int64)
    rows = np.array([r for c in cols for r in sorted(c)], np.int32)
    res = api.reduce(torch.as_tensor(cp, device=gpu), torch.as_tensor(rows, device=gpu),
                     torch.as_tensor(np.asarray(dim, np.int8), device=gpu))
    want = oracle.reduce_twist(cp, rows, np.asarray(dim, np.int8))
    assert np.array_equal(res.low_star.cpu().numpy(), want) and res.rounds == 1
    api.selftest(gpu)


def test_instances_of_a_callers_matrix(gpu):
    """``reduce`` and ``reduce_filtration`` pass instance offsets on, to the
    results of ``reduce_batched``; the allocation-free entry point takes none."""
    rng = np.random.default_rng(17)
    f, off = api.build_vr([torch.as_tensor(rng.integers(0, 99, (n, 3)).astype(np.int32), device=gpu) for n in (9, 0, 14)])
    want = api.reduce_batched(f, off)
    t = f.to_torch()
    dev_off = torch.as_tensor(off, dtype=torch.int64, device=gpu)
    for got in (api.reduce(t["col_ptr"], t["rows"], t["dim"], inst_col_off=dev_off),
                api.reduce_filtration(f, inst_col_off=dev_off)):
        for k in ("low_star", "pair_birth", "pair_death", "essential", "inst_pair_off", "inst_ess_off", "pair_inst"):
            assert torch.equal(getattr(got, k), getattr(want, k)), k
    for call in (lambda: api.reduce(t["col_ptr"], t["rows"], t["dim"], inst_col_off=dev_off, noalloc=True),
                 lambda: api.reduce_filtration(f, inst_col_off=dev_off, noalloc=True),
                 lambda: api.reduce_batched(f, off, noalloc=True)):
        with pytest.raises(ValueError):
            call()


@pytest.mark.parametrize("dtype", [torch.int32, torch.float32])
def test_a_batch_of_empty_clouds(gpu, dtype):
    """An empty filtration, in a new object as in a kept one, and no error left
    behind for the next call."""
    empty = [torch.zeros((0, 3), dtype=dtype, device=gpu)] * 2
    kept, _ = api.build_vr(torch.arange(6, device=gpu).reshape(3, 2).to(dtype))
    for out in (None, kept):
        f, off = api.build_vr(empty, out=out)
        assert f.m == 0 and off == [0, 0, 0] and f.to_torch()["col_ptr"].tolist() == [0]
        assert api.reduce_batched(f, off).low_star.numel() == 0
        assert api.build_vr(torch.arange(6, device=gpu).reshape(3, 2).to(dtype), out=f)[0].m == 7


@pytest.mark.parametrize("n,D,count", [(40, 335, 1), (40, 337, 1), (40, 340, 30), (90, 500, 3), (181, 20, 2), (190, 16, 2)])
@pytest.mark.parametrize("f32", [False, True])
def test_clouds_of_many_coordinates(gpu, n, D, count, f32):
    """Either side of the line from which one workgroup's distances are too many
    (2^18 coordinates of a cloud's pairs, and more in a batch)."""
    rng = np.random.default_rng(n + D)
    clouds = [rng.normal(size=(n, D)) for _ in range(count)]
    clouds = [c.astype(np.float32) if f32 else np.rint(c * 999).astype(np.int32) for c in clouds]
    maxdim = 2 if n < 100 else 1
    f, off = api.build_vr([torch.as_tensor(c, device=gpu) for c in clouds], None, maxdim)
    t = f.to_torch()
    low = api.reduce_batched(f, off).low_star.cpu().numpy()
    for c, a, b in zip(clouds, off, off[1:]):
        ref = (oracle.build_vr_f32 if f32 else oracle.build_vr_i32)(c, maxdim=maxdim)
        s, e = int(t["col_ptr"][a]), int(t["col_ptr"][b])
        assert b - a == ref.m and np.array_equal(t["rows"][s:e].cpu().numpy(), ref.rows + a)
        assert np.array_equal(t["value"][a:b].cpu().numpy().astype(np.float64), ref.value.astype(np.float64))
        want = oracle.reduce_twist(ref.col_ptr, ref.rows, ref.dim)
        assert np.array_equal(low[a:b], np.where(want >= 0, want + a, -1))
