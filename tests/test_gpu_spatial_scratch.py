"""How much scratch a two-pass spatial search asks for: the room to keep rows only
where they would be kept, and no more than the least where that does not fit the
device memory (forced here by an allocator that refuses it)."""
import ctypes as C

import pytest
import torch

from paper_1908_11807_amd import abx, datagen

pytestmark = pytest.mark.gpu

N, M = 20_000, 30_000


def points(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand((n, 3), generator=g, device="cuda")


@pytest.fixture
def setup():
    t = abx.bvh_build(points(N, 1), node_format="q16")
    q = points(M, 2)
    radius = float(datagen.radius_for_density(N, 10))
    pr = abx.Predicates(abx.PRED_WITHIN, q.data_ptr(), M, None, radius, 1)
    least, full = C.c_size_t(), C.c_size_t()
    assert abx.library().abx_query_spatial_sizes_for(t.handle, C.byref(pr), 0, C.byref(least),
                                                     C.byref(full)) == abx.OK
    return t, q, radius, least.value, full.value


def sizes_for(t, q, radius, capacity):
    pr = abx.Predicates(abx.PRED_WITHIN, q.data_ptr(), M, None, radius, 1)
    b = C.c_size_t()
    assert abx.library().abx_query_spatial_sizes_for(t.handle, C.byref(pr), capacity, None,
                                                     C.byref(b)) == abx.OK
    return b.value


def test_sizes(setup):
    t, q, radius, least, full = setup
    assert 100 * M < full - least < 200 * M
    assert sizes_for(t, q, radius, 24 * M) == full
    assert sizes_for(t, q, radius, 24 * M + 1) == least      # rows expected longer
    assert sizes_for(t, q, 4 * radius, 0) == least
    pr = abx.Predicates(abx.PRED_WITHIN, q.data_ptr(), M, None, radius, 1)
    L = abx.library()
    assert L.abx_query_spatial_sizes_for(t.handle, C.byref(pr), -1, None, None) == abx.ERR_INVALID_ARG
    assert L.abx_query_spatial_sizes_for(None, C.byref(pr), 0, None, None) == abx.ERR_INVALID_ARG


@pytest.mark.parametrize("capacity", [None, 15 * M])
def test_search_without_room_for_kept_rows(setup, capacity, monkeypatch):
    t, q, radius, least, full = setup
    want = abx.query_spatial(t, q, radius=radius, capacity=capacity)
    asked = []
    allocate = abx._bytes

    def small(n, device):
        asked.append(n)
        if n > least:
            raise torch.OutOfMemoryError("refused")
        return allocate(n, device)

    monkeypatch.setattr(abx, "_bytes", small)
    off, idx = abx.query_spatial(t, q, radius=radius, capacity=capacity)
    assert asked == [full, least]
    assert torch.equal(off, want[0]) and torch.equal(idx, want[1])


def test_stats_and_long_rows_take_the_least(setup, monkeypatch):
    t, q, radius, least, full = setup
    want = abx.query_spatial_stats(t, q, radius=radius)
    asked = []
    allocate = abx._bytes
    monkeypatch.setattr(abx, "_bytes", lambda n, device: asked.append(n) or allocate(n, device))
    assert torch.equal(abx.query_spatial_stats(t, q, radius=radius), want)
    abx.query_spatial(t, q, radius=radius, capacity=40 * M)
    assert asked == [least, least]
