"""The boxes of forests of few points, whose chunks are as long as a share of one
CU: the points that span a tree stand at the edges of those chunks (of every
length the sizes lead to), and many small trees do not queue in a few
workgroups (512 sets of 3 to 30 points took 45 times as long as one set of the
same points)."""
import numpy as np
import pytest
import torch

from paper_1908_11807_amd import abx

pytestmark = pytest.mark.gpu


def chunk(n):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return min(max(n // cus, 256), 16384)


@pytest.mark.parametrize("sizes", [[255, 1], [256, 257, 0, 1], [100_000], [1] * 300 + [70_001, 2],
                                   [300_000, 5, 300_000]])
def test_extreme_points_at_chunk_edges(sizes):
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    rng = np.random.default_rng(n)
    pts = rng.integers(0, 50, size=(n, 3)).astype(np.float32)
    c = chunk(n)
    edges = [i for i in (0, c - 1, c, 2 * c - 1, n // c * c - 1, n - 1) if 0 <= i < n]
    for j, i in enumerate(edges):
        pts[i, j % 3] = (-1) ** j * (100 + 10 * j)
    qo = np.arange(len(sizes) + 1) * 2
    q = rng.integers(-120, 170, size=(int(qo[-1]), 3)).astype(np.float32)
    plan = abx.ForestPlan(torch.from_numpy(pts).cuda(), off.tolist(), torch.from_numpy(q).cuda(),
                          qo.tolist(), 5, node_format="q16")
    o, ki, kd = (x.cpu().numpy() for x in plan.run())
    for t in range(len(sizes)):
        own = pts[off[t]:off[t + 1]].astype(np.int64)
        for j in range(qo[t], qo[t + 1]):
            d2 = ((own - q[j].astype(np.int64)) ** 2).sum(1)
            want = np.argsort(d2, kind="stable")[:5]
            assert np.array_equal(ki[o[j]:o[j + 1]], want), (t, j)
            assert np.array_equal(kd[o[j]:o[j + 1]], np.sqrt(d2[want].astype(np.float32))), (t, j)


def test_many_small_trees():
    sizes = np.linspace(3, 30, 512).astype(int)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    pts = torch.rand((n, 3), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")

    def ms(offsets):
        plan = abx.ForestPlan(pts, offsets, pts, offsets, 1, node_format="q16")
        plan.build()
        best = float("inf")
        for _ in range(4):
            abx.timing_enable(True)
            abx.timing_reset()
            plan.build()
            torch.cuda.synchronize()
            best = min(best, abx.timing_get("forest_boxes")[0])
            abx.timing_enable(False)
        return best

    many, one = ms(off), ms(np.array([0, n], np.int64))
    print(f"512 sets {1e3 * many:.1f} us, one {1e3 * one:.1f} us", flush=True)
    assert many < 20.0 * one
