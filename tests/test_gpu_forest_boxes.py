"""The boxes of a forest's trees, with the points that span them at the edges
of the chunks that are reduced together, and trees of no point, one and a few
between long ones.  The quantised node grid is that of all the boxes, and a
tree of one point is answered from its box alone, so a bound that a chunk
loses shows in the rows; these are exact (small integers)."""
import numpy as np
import pytest
import torch

from paper_1908_11807_amd import abx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[40_000], [16_383, 1, 16_384, 0, 3, 16_385, 1, 1],
                                   [1] * 70 + [16_384 * 2 + 5] + [2] * 5])
@pytest.mark.parametrize("fmt", ["fp32", "q16"])
def test_extreme_points_at_chunk_edges(sizes, fmt):
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    rng = np.random.default_rng(n)
    pts = rng.integers(0, 50, size=(n, 3)).astype(np.float32)
    edges = [i for i in (0, 16_383, 16_384, 32_767, 32_768, n - 1) if i < n]
    for j, i in enumerate(edges):
        pts[i, j % 3] = (-1) ** j * (100 + 10 * j)
    qo = np.arange(len(sizes) + 1) * 4
    q = rng.integers(-120, 170, size=(int(qo[-1]), 3)).astype(np.float32)
    plan = abx.ForestPlan(torch.from_numpy(pts).cuda(), off.tolist(), torch.from_numpy(q).cuda(),
                          qo.tolist(), 5, node_format=fmt)
    o, ki, kd = (x.cpu().numpy() for x in plan.run())
    for t in range(len(sizes)):
        own = pts[off[t]:off[t + 1]].astype(np.int64)
        for j in range(qo[t], qo[t + 1]):
            d2 = ((own - q[j].astype(np.int64)) ** 2).sum(1)
            want = np.argsort(d2, kind="stable")[:5]
            assert np.array_equal(ki[o[j]:o[j + 1]], want), (t, j)
            assert np.array_equal(kd[o[j]:o[j + 1]], np.sqrt(d2[want].astype(np.float32))), (t, j)
