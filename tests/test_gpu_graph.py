"""The blocks reduced as graphs (edges over vertices; top simplices over
their faces when no face has more than two cofaces) against the oracle: edges
with fewer or more than two vertices, faces with none, one, two and more
cofaces, long walks, and volumes one or two cells thin."""
import numpy as np
import pytest
import torch

import oracle
from paper_1708_04710_amd import api, synth
from tests import brute

pytestmark = pytest.mark.gpu


def _check(cols, dim, gpu):
    cp = np.cumsum([0] + [len(c) for c in cols]).astype(np.int64)
    rows = np.array([r for c in cols for r in sorted(c)], np.int32)
    dim = np.asarray(dim, np.int8)
    want = oracle.reduce_standard(cp, rows)
    res = api.reduce(torch.as_tensor(cp, device=gpu), torch.as_tensor(rows, device=gpu),
                     torch.as_tensor(dim, device=gpu))
    assert np.array_equal(res.low_star.cpu().numpy(), want)
    b, d = oracle.pairs(want)
    assert np.array_equal(res.pair_birth.cpu().numpy(), b) and np.array_equal(res.pair_death.cpu().numpy(), d)
    assert np.array_equal(res.essential.cpu().numpy(), oracle.essential(want))
    return res


def test_quotient_complexes(gpu):
    """K modulo a subcomplex: edges lose vertices, triangles edges."""
    rng = np.random.default_rng(31)
    for _ in range(60):
        cp, rows, dim, _, _ = brute.random_filtration(rng, n_vertices=int(rng.integers(3, 10)),
                                                      n_facets=int(rng.integers(2, 10)), max_dim=int(rng.integers(1, 4)))
        m = len(dim)
        faces = [list(rows[cp[j]:cp[j + 1]]) for j in range(m)]
        gone = np.zeros(m, bool)
        for j in rng.choice(m, size=min(m, int(rng.integers(1, 4))), replace=False):
            stack = [int(j)]
            while stack:
                k = stack.pop()
                gone[k] = True
                stack += [int(r) for r in faces[k] if not gone[r]]
        new = np.cumsum(~gone) - 1
        keep = np.flatnonzero(~gone)
        _check([[int(new[r]) for r in faces[j] if not gone[r]] for j in keep], dim[keep], gpu)


@pytest.mark.parametrize("most", [1, 2, 5])
def test_edges_of_any_length(gpu, most):
    rng = np.random.default_rng(most)
    nv, ne = 300, 700
    cols = [[] for _ in range(nv)]
    cols += [list(rng.choice(nv, size=int(rng.integers(0, most + 1)), replace=False)) for _ in range(ne)]
    _check(cols, [0] * nv + [1] * ne, gpu)


@pytest.mark.parametrize("pages", [1, 2, 3, 4])
def test_a_book_of_triangles(gpu, pages):
    """`pages` triangles on one edge (a graph up to two), with enough free
    edges that the counts alone do not decide."""
    nv = 40
    verts = [[] for _ in range(nv)]
    ends = [(0, 1)] + [(a, 2 + p) for p in range(pages) for a in (0, 1)] + [(k, k + 1) for k in range(6, nv - 1)]
    edges = [[a, b] for a, b in ends]
    tris = [[nv, nv + 1 + 2 * p, nv + 2 + 2 * p] for p in range(pages)]
    _check(verts + edges + tris, [0] * nv + [1] * len(edges) + [2] * pages, gpu)


def test_long_paths_in_random_order(gpu):
    """A path whose edges come in random order (its last edges join halves
    thousands of vertices long) and a strip of triangles likewise."""
    rng = np.random.default_rng(7)
    n = 6000
    e = rng.permutation(n - 1)
    res = _check([[] for _ in range(n)] + [[int(k), int(k) + 1] for k in e], [0] * n + [1] * (n - 1), gpu)
    assert res.pair_birth.numel() == n - 1
    k = 3000  # strip: vertices 0..k+1, edges (i, i+1), (i, i+2), triangles (i, i+1, i+2)
    pairs = [(i, i + 1) for i in range(k + 1)] + [(i, i + 2) for i in range(k)]
    order = rng.permutation(len(pairs))
    at = {pairs[int(o)]: k + 2 + p for p, o in enumerate(order)}
    tri = rng.permutation(k)
    cols = [[] for _ in range(k + 2)] + [list(pairs[int(o)]) for o in order]
    cols += [[at[(int(i), int(i) + 1)], at[(int(i) + 1, int(i) + 2)], at[(int(i), int(i) + 2)]] for i in tri]
    _check(cols, [0] * (k + 2) + [1] * len(pairs) + [2] * k, gpu)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 50), (1, 23, 31), (2, 17, 19), (9, 1, 14)])
@pytest.mark.parametrize("ties", [False, True])
def test_thin_volumes(gpu, shape, ties):
    g = synth.random_grid(3, shape, ties=ties)
    f = api.build_lowerstar(torch.as_tensor(g, device=gpu))
    ref = oracle.build_lowerstar(g)
    res = api.reduce_filtration(f)
    assert np.array_equal(res.low_star.cpu().numpy(), oracle.reduce_twist(ref.col_ptr, ref.rows, ref.dim))
