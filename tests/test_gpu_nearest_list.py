"""The nearest walk's candidate lists, one size per register list and the ends
of the range each serves, on integer lattices: every squared distance is an
exact small integer, so the expected rows (distance, then index) follow from
integer arithmetic alone, with no tolerance.  Points are repeated, so rows
hold zero distances and long ties that only the index orders; queries with an
infinite coordinate put every point at infinity."""
import numpy as np
import pytest
import torch

from paper_1908_11807_amd import abx

pytestmark = pytest.mark.gpu


def rows(pts, q, k):
    d2 = ((q[:, None, :].astype(np.int64) - pts[None].astype(np.int64)) ** 2).sum(-1)
    order = np.argsort(d2, axis=1, kind="stable")[:, :k]
    return order.astype(np.int32), np.take_along_axis(d2, order, 1)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 10, 11, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("fmt", ["fp32", "q16", "q16w"])
def test_lists_order_ties_and_zeros(k, fmt):
    rng = np.random.default_rng(k)
    pts = rng.integers(0, 9, size=(1500, 3)).astype(np.float32)
    pts = np.concatenate([pts, pts[:700]])             # exact repeats
    q = np.concatenate([pts[rng.integers(0, 2200, 40)],  # on a point: zero distances
                        rng.integers(-3, 12, size=(60, 3)).astype(np.float32)])
    t = abx.bvh_build(torch.from_numpy(pts).cuda(), node_format=fmt)
    _, ki, kd = abx.query_nearest(t, torch.from_numpy(q).cuda(), k)
    want, d2 = rows(pts, q, k)
    assert np.array_equal(ki.cpu().numpy(), want)
    # float32 square root, correctly rounded
    assert np.array_equal(kd.cpu().numpy(), np.sqrt(d2.astype(np.float32)))
    inf = torch.full((3, 3), float("inf"), device="cuda")
    inf[1, 1:] = 2.0
    inf[2] = -float("inf")
    _, ki, kd = abx.query_nearest(t, inf, k)
    assert np.array_equal(ki.cpu().numpy(), np.tile(np.arange(k, dtype=np.int32), (3, 1)))
    assert bool(torch.isinf(kd).all())
