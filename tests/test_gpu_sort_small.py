"""Sorts of one workgroup (up to 12 288 pairs) and the first sizes beyond, over
the remainders of a wavefront's share and of the last digit, with and without
values.  Whole numbers: equal to a stable argsort."""
import numpy as np
import pytest
import torch

from paper_1908_11807_amd import abx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 64, 65, 1023, 1024, 1025, 2049, 12_287, 12_288, 12_289])
@pytest.mark.parametrize("key_bits", [1, 8, 17, 32, 33, 64])
def test_small_sorts_are_stable(n, key_bits):
    rng = np.random.default_rng(n + key_bits)
    keys = rng.integers(0, 2 ** key_bits, size=n, dtype=np.uint64, endpoint=False) \
        if key_bits < 64 else rng.integers(0, 2 ** 64, size=n, dtype=np.uint64)
    keys[rng.integers(0, n, n // 2)] = keys[0]                  # repeats
    keys[rng.integers(0, n, n // 8 + 1)] = np.uint64(2 ** key_bits - 1)
    dev = keys.astype(np.uint32).view(np.int32) if key_bits <= 32 else keys.view(np.int64)
    vals = rng.integers(-2 ** 31, 2 ** 31, size=n).astype(np.int32)
    perm = np.argsort(keys, kind="stable")
    for v, want in ((None, perm), (torch.from_numpy(vals).cuda(), vals[perm])):
        ko, vo = abx.radix_sort_pairs(torch.from_numpy(dev).cuda(), key_bits, vals=v)
        assert np.array_equal(ko.cpu().numpy(), dev[perm])
        assert np.array_equal(vo.cpu().numpy(), want)
