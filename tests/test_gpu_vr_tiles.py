"""The edge-order builder where its tiles can go wrong: points around the limit
and the words of a cloud whose ranks fit LDS, edges around a workgroup's share,
few edges and the many from which the ranks are held there, and clouds that are
views of other tensors."""
import numpy as np
import pytest
import torch

from paper_1708_04710_amd import api
from tests.test_gpu_vr_edges import _same_as_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("edges", [1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1024])
def test_edges_around_a_share(gpu, edges):
    p = np.random.default_rng(edges).integers(0, 1 << 14, (60, 2)).astype(np.int32)
    d = ((p[:, None].astype(np.int64) - p[None]) ** 2).sum(2)[np.triu_indices(60, 1)]
    _same_as_oracle([p], [int(np.sort(d)[edges - 1])], 2, gpu)


@pytest.mark.parametrize("n,count,pct", [(256, 22, 0.1), (257, 22, 0.1), (64, 40, 1.0), (65, 40, 1.0), (33, 130, 1.0)])
@pytest.mark.parametrize("side", [1 << 14, 60])
def test_many_edges(gpu, n, count, pct, side):
    """More than 2^16 edges in all, without and with edges of equal value."""
    rng = np.random.default_rng(n)
    clouds = [rng.integers(0, side, (n - int(rng.integers(0, 3)) * (k > 0), 2)).astype(np.int32) for k in range(count)]
    thrs = [-1 if pct == 1.0 else int(side * side * 2 * pct) for _ in clouds]
    _same_as_oracle(clouds, thrs, 2, gpu)


def test_clouds_that_are_views(gpu):
    rng = np.random.default_rng(9)
    wide = torch.as_tensor(rng.normal(size=(40, 7)).astype(np.float32), device=gpu)
    tall = torch.as_tensor(rng.normal(size=(3, 33)).astype(np.float32), device=gpu)
    views = [wide[:, 2:5], tall.t(), wide[1::2], wide[5:9], wide[:0], tall.t()[3:], wide[7], wide[3:30, :1]]
    views[6] = views[6].reshape(7, 1)
    thr = [-1.0] * len(views)
    f, off = api.build_vr(views, thr, 2)
    g, want = api.build_vr([v.clone(memory_format=torch.contiguous_format) for v in views], thr, 2)
    assert off == want
    a, b = f.to_torch(), g.to_torch()
    assert all(torch.equal(a[k], b[k]) for k in a)
    with pytest.raises((RuntimeError, ValueError)):
        api.build_vr([wide, wide.cpu()], thr[:2], 2)


@pytest.mark.parametrize("edges", [1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 16383, 16384, 16385])
def test_edges_around_a_sort(gpu, edges):
    """One, two, four, eight and sixteen keys a thread, and the device-wide sort."""
    p = np.random.default_rng(edges).integers(0, 1 << 14, (190, 4)).astype(np.int32)
    d = ((p[:, None].astype(np.int64) - p[None]) ** 2).sum(2)[np.triu_indices(190, 1)]
    _same_as_oracle([p], [int(np.sort(d)[edges - 1])], 1, gpu)
