"""Row offsets over the sizes that decide how the counts are scanned: inside and
across a tile of 4096, a group of four cut short, and either side of 4096
tiles.  One point and radii that hit or miss it, so the counts are known."""
import pytest
import torch

from paper_1908_11807_amd import abx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 3, 1023, 1025, 4095, 4096, 4097, 12_290, 4096 * 4096,
                               4096 * 4096 + 1, 4096 * 4096 + 4098])
def test_offsets_are_the_running_sum(m):
    t = abx.bvh_build(torch.zeros(1, 3, device="cuda"))
    i = torch.arange(m, device="cuda")
    hit = ((i * 7919) % 13 < 5) | (i == m - 1)
    q = torch.ones(m, 3, device="cuda")
    off, idx = abx.query_spatial(t, q, radii=torch.where(hit, 2.0, 1.0).float(), sort_queries=False)
    want = torch.cumsum(hit.int(), 0, dtype=torch.int32)
    assert off[0].item() == 0 and torch.equal(off[1:], want)
    assert idx.numel() == int(want[-1]) and not bool(idx.any())
