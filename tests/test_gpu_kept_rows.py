"""The two-pass spatial search with rows kept by its first pass: rows of every
length around the limits (kept slots, extensions, the pool of extensions) equal,
in order, those of the search that walks twice (a capacity far above the
results asks for it), whichever way the second pass is reached."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1908_11807_amd import abx, datagen

pytestmark = pytest.mark.gpu

# sites of so many equal points each: a query on a site finds them all
LENGTHS = [0, 1, 7, 8, 9, 31, 32, 33, 40, 63, 64, 65, 95, 96, 127, 128, 129, 200, 500]


def sites(lengths, seed):
    rng = np.random.default_rng(seed)
    at = np.stack(np.unravel_index(rng.permutation(8000)[:len(lengths)], (20, 20, 20)), 1)
    at = at.astype(np.float32)
    pts = np.repeat(at, lengths, axis=0)
    return at, np.ascontiguousarray(pts[rng.permutation(len(pts))])


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def base_bytes(t, pr, m):
    b = C.c_size_t()
    L = abx.library()
    assert L.abx_query_spatial_1p_sizes(t.handle, C.byref(pr), 1, C.byref(b)) == abx.OK
    return b.value - 256 - -(-m * 4 // 256) * 256


def call(t, q, kind, capacity, scratch_bytes=None, one_pass=0, radius=0.25):
    """(offsets, indices) through the C entry points: the search, then the fill
    if the capacity was too small; one_pass: that scheme first."""
    L = abx.library()
    m = q.shape[0]
    pr = abx.Predicates(kind, q.data_ptr(), m, None, radius, 1)
    b = C.c_size_t()
    if one_pass:
        assert L.abx_query_spatial_1p_sizes(t.handle, C.byref(pr), one_pass, C.byref(b)) == abx.OK
    else:
        assert L.abx_query_spatial_sizes(t.handle, C.byref(pr), C.byref(b)) == abx.OK
    n = b.value if scratch_bytes is None else scratch_bytes
    sc = torch.full((n,), 0x5a, dtype=torch.uint8, device="cuda")
    off = torch.empty(m + 1, dtype=torch.int32, device="cuda")
    idx = torch.full((max(capacity, 1),), -7, dtype=torch.int32, device="cuda")
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    vp = C.c_void_p
    if one_pass:
        info = torch.zeros(2, dtype=torch.int32, device="cuda")
        assert L.abx_query_spatial_1p(t.handle, C.byref(pr), one_pass, vp(sc.data_ptr()), n,
                                      vp(off.data_ptr()), vp(idx.data_ptr()), 1, vp(info.data_ptr()),
                                      s) == abx.OK
        assert int(info[0]) == abx.ERR_CAPACITY
        total = int(off[-1])
    else:
        tot = C.c_int64()
        st = L.abx_query_spatial(t.handle, C.byref(pr), vp(sc.data_ptr()), n, vp(off.data_ptr()),
                                 vp(idx.data_ptr()) if capacity else None, capacity, C.byref(tot), s)
        total = tot.value
        if st == abx.OK:
            return off, idx[:total]
        assert st == abx.ERR_CAPACITY
    idx = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    assert L.abx_query_spatial_fill(t.handle, C.byref(pr), vp(sc.data_ptr()), n, vp(off.data_ptr()),
                                    vp(idx.data_ptr()), total, s) == abx.OK
    return off, idx


@pytest.mark.parametrize("fmt", ["fp32", "q16", "q16w"])
@pytest.mark.parametrize("boxes", [False, True])
@pytest.mark.parametrize("m", [1, 65, 1500])
def test_kept_rows_equal_walked_rows(fmt, boxes, m):
    lengths = np.array(LENGTHS * 8)
    at, pts = sites(lengths, m)
    prims = datagen.boxes_around(pts, 5, 0.1) if boxes else pts
    t = abx.bvh_build(dev(prims), kind=int(boxes), node_format=fmt)
    pick = np.random.default_rng(m).integers(0, len(at), m)
    q = at[pick]
    kind = abx.PRED_WITHIN
    if boxes:
        kind = abx.PRED_INTERSECTS_BOX
        q = np.concatenate([q - 0.2, q + 0.2], axis=1).astype(np.float32)
    q = dev(q)
    total = int(lengths[pick].sum())
    want = call(t, q, kind, max(total, 24 * m + 1))        # walked twice
    assert np.array_equal(np.diff(want[0].cpu().numpy()), lengths[pick])
    pr = abx.Predicates(kind, q.data_ptr(), m, None, 0.25, 1)
    for got in (call(t, q, kind, 0),                         # kept rows, by the fill
                call(t, q, kind, total if total <= 24 * m else 0),
                call(t, q, kind, 0, scratch_bytes=base_bytes(t, pr, m)),   # no room to keep
                call(t, q, kind, 0, one_pass=4) if total > 1 else want):
        assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


def test_pool_of_extensions_runs_out():
    # every row asks for an extension, one in sixteen gets it
    at, pts = sites(np.array([50] * 30), 3)
    t = abx.bvh_build(dev(pts), node_format="q16")
    q = dev(at[np.random.default_rng(4).integers(0, 30, 20_000)])
    want = call(t, q, abx.PRED_WITHIN, 50 * 20_000)          # capacity above 24 a query: walked twice
    got = call(t, q, abx.PRED_WITHIN, 0)
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])
    off, idx = abx.query_spatial(t, q, radius=0.25, sort_queries=False)
    assert torch.equal(want[0], off) and torch.equal(want[1], idx)


@pytest.mark.parametrize("fmt", ["fp32", "q16w"])
@pytest.mark.parametrize("buffer", [1, 7, 8, 9, 16, 23, 64])
def test_one_pass_rows_end_anywhere(fmt, buffer):
    # rows of 0 to 40 hits against buffers that end inside, at and beyond a
    # group of eight: stored rows, and the second walk after an overflow, equal
    # the two-pass rows entry for entry
    pts = torch.arange(41, dtype=torch.float32, device="cuda")[:, None].repeat(1, 3) * 0.01
    q = torch.zeros(200, 3, device="cuda")
    radii = torch.arange(200, dtype=torch.float32, device="cuda") * (0.01 * 3 ** 0.5 * 0.21)
    t = abx.bvh_build(pts, node_format=fmt)
    off, idx = abx.query_spatial(t, q, radii=radii)
    assert {int(c) for c in (off[1:] - off[:-1])} >= set(range(1, 41))
    o1, x1, _ = abx.query_spatial_1p(t, q, buffer, radii=radii)
    assert torch.equal(o1, off) and torch.equal(x1[:idx.numel()], idx)
