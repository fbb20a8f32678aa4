"""Nearest queries kept on their lanes: with the visit budget off, no query of a
batch is handed to a workgroup, so the rows below come from the register lists
alone, one list size and the ends of its range at a time.  Integer lattices
with repeated points: the expected rows (distance, then index) follow from
integer arithmetic, with no tolerance.  Queries with an infinite coordinate put
every point at infinity, where the index alone orders a row, after a walk of the
whole tree."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1908_11807_amd import abx

pytestmark = pytest.mark.gpu

VP = C.c_void_p


def rows(pts, q, k):
    d2 = ((q[:, None, :].astype(np.int64) - pts[None].astype(np.int64)) ** 2).sum(-1)
    order = np.argsort(d2, axis=1, kind="stable")[:, :k]
    return order.astype(np.int32), np.sqrt(np.take_along_axis(d2, order, 1).astype(np.float32))


def search(t, q, k):
    """(indices, distances, queries handed over): the count of the handed-over
    queries is the first word behind the scratch's four arrays of one word a query."""
    L = abx.library()
    m = q.shape[0]
    b = C.c_size_t()
    assert L.abx_query_nearest_sizes(t.handle, m, k, C.byref(b)) == abx.OK
    sc = torch.zeros(b.value, dtype=torch.uint8, device="cuda")
    off = torch.empty(m + 1, dtype=torch.int32, device="cuda")
    idx = torch.empty((m, k), dtype=torch.int32, device="cuda")
    dist = torch.empty((m, k), dtype=torch.float32, device="cuda")
    s = VP(torch.cuda.current_stream().cuda_stream)
    assert L.abx_query_nearest(t.handle, VP(q.data_ptr()), m, k, 1, VP(sc.data_ptr()), b.value,
                               VP(off.data_ptr()), VP(idx.data_ptr()), VP(dist.data_ptr()),
                               s) == abx.OK
    at = 4 * (-(-4 * m // 256) * 256)
    handed = int(sc[at:at + 4].view(torch.int32).item())
    return idx.cpu().numpy(), dist.cpu().numpy(), handed


@pytest.fixture(params=[0, -1])
def no_budget(request):
    old = abx.set_nearest_budget(request.param)
    yield
    abx.set_nearest_budget(old)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 10, 11, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("fmt", ["fp32", "q16", "q16w"])
def test_lists_of_one_lane(k, fmt, no_budget):
    rng = np.random.default_rng(k)
    pts = rng.integers(0, 9, size=(1500, 3)).astype(np.float32)
    pts = np.concatenate([pts, pts[:700]])
    q = np.concatenate([pts[rng.integers(0, 2200, 40)],
                        rng.integers(-3, 12, size=(60, 3)).astype(np.float32)])
    want, dist = rows(pts, q, k)
    far = np.full((3, 3), np.inf, np.float32)
    far[1, 1:] = 2.0
    far[2] = -np.inf
    t = abx.bvh_build(torch.from_numpy(pts).cuda(), node_format=fmt)
    ki, kd, handed = search(t, torch.from_numpy(np.concatenate([q, far])).cuda(), k)
    assert handed == 0
    assert np.array_equal(ki[:100], want) and np.array_equal(kd[:100], dist)
    assert np.array_equal(ki[100:], np.tile(np.arange(k, dtype=np.int32), (3, 1)))
    assert np.isinf(kd[100:]).all()


def test_a_budget_hands_queries_over():
    # (so the word read above is the count)
    pts = np.random.default_rng(1).integers(0, 9, size=(2200, 3)).astype(np.float32)
    t = abx.bvh_build(torch.from_numpy(pts).cuda())
    q = torch.from_numpy(pts[:101]).cuda()
    old = abx.set_nearest_budget(1)
    try:
        assert search(t, q, 10)[2] == 101
    finally:
        assert abx.set_nearest_budget(old) == 1
