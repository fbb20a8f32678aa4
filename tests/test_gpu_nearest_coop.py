"""Nearest queries answered by whole workgroups, over the sizes that decide the
workgroup (a query for each CU, more, many), the node formats, lists that are
resumed and lists that start over, and walks long enough to be passed on to the
largest workgroups.  Lattice points and repeated points: every squared distance
is an exact small integer, so the expected rows (distance, then index) follow
from integer arithmetic, with no tolerance."""
import numpy as np
import pytest
import torch

from paper_1908_11807_amd import abx

pytestmark = pytest.mark.gpu


def rows(pts, q, k):
    d2 = ((q[:, None, :].astype(np.int64) - pts[None].astype(np.int64)) ** 2).sum(-1)
    order = np.argsort(d2, axis=1, kind="stable")[:, :k]
    return order.astype(np.int32), np.sqrt(np.take_along_axis(d2, order, 1).astype(np.float32))


@pytest.fixture
def budget():
    old = abx.set_nearest_budget(8192)
    yield abx.set_nearest_budget
    abx.set_nearest_budget(old)


@pytest.mark.parametrize("m", [1, 256, 257, 4097])
@pytest.mark.parametrize("fmt", ["fp32", "q16", "q16w"])
def test_rows_do_not_depend_on_the_workgroup(fmt, m, budget):
    rng = np.random.default_rng(m)
    pts = rng.integers(0, 13, size=(3000, 3)).astype(np.float32)
    q = rng.integers(-4, 17, size=(m, 3)).astype(np.float32)
    t = abx.bvh_build(torch.from_numpy(pts).cuda(), node_format=fmt)
    want, dist = rows(pts, q, 64)
    for k in (1, 10, 32, 33, 64):
        for visits in (1, 9, 60):
            budget(visits)
            _, ki, kd = abx.query_nearest(t, torch.from_numpy(q).cuda(), k)
            assert np.array_equal(ki.cpu().numpy(), want[:, :k]), (k, visits)
            assert np.array_equal(kd.cpu().numpy(), dist[:, :k]), (k, visits)


@pytest.mark.parametrize("m", [2, 300, 4200])
@pytest.mark.parametrize("fmt", ["fp32", "q16w"])
def test_ties_over_the_whole_tree(fmt, m):
    # every point at the same distance: no node can be skipped, the candidates
    # outnumber any list, and the index alone orders them
    pts = torch.ones(400_003, 3, device="cuda")
    q = torch.zeros(m, 3, device="cuda")
    q[:, 0] = 1.0
    t = abx.bvh_build(pts, node_format=fmt)
    for k in (3, 40):
        _, ki, kd = abx.query_nearest(t, q, k)
        assert bool((ki == torch.arange(k, dtype=torch.int32, device="cuda")).all())
        assert bool((kd == 2.0 ** 0.5).all())


def test_forest_rows_do_not_depend_on_the_workgroup():
    rng = np.random.default_rng(5)
    sizes, qs = [2500, 1, 200_001], [300, 5, 40]
    pts = rng.integers(0, 13, size=(sum(sizes), 3)).astype(np.float32)
    pts[2501:] = 1.0                                    # ties over a whole tree
    q = rng.integers(-4, 17, size=(sum(qs), 3)).astype(np.float32)
    q[305:] = (1.0, 0.0, 0.0)
    po, qo = np.concatenate([[0], np.cumsum(sizes)]), np.concatenate([[0], np.cumsum(qs)])
    k = 12
    plan = abx.ForestPlan(torch.from_numpy(pts).cuda(), po.tolist(), torch.from_numpy(q).cuda(),
                          qo.tolist(), k)
    plan.build()
    for visits in (1, 9, 60, 16384):
        plan.query(dict(blocks_per_cu=4, tiles_per_grab=1, budget=visits))
        off, ki, kd = (x.cpu().numpy() for x in plan.results())
        for i in (0, 1, 2):
            for j in range(qo[i], qo[i + 1], 1 if i < 2 else 20):
                want, dist = rows(pts[po[i]:po[i + 1]], q[j:j + 1], k)
                assert np.array_equal(ki[off[j]:off[j + 1]], want[0]), (visits, i, j)
                assert np.array_equal(kd[off[j]:off[j + 1]], dist[0]), (visits, i, j)
