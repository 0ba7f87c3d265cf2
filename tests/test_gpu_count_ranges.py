"""GPU parity of interval counting for key spaces beyond one block's LDS: one to 32 ranges and
past them, intervals that are one part, several parts or empty, most requests in one of many
intervals, intervals across the bounds by which items are numbered, streams that start off a
16-byte boundary, out-of-range keys. Reference: numpy.bincount per interval."""
import numpy as np
import pytest
import torch

from paper_2608_19677_amd import binding as B

from cr_check import say

pytestmark = pytest.mark.gpu

CASES = [
    # K, interval sizes, first key's offset in words, bad keys
    (40_900, [10_000, 0, 1, 70_001], 0, False), (41_000, [131_072, 131_073, 5], 1, False), (81_801, [400_003], 2, True),
    (128_824, [1] * 30 + [600_000] + [0] * 5 + [17], 3, False), (1_000_000, [200_000, 300_001], 1, True),
    (1_300_000, [50_000, 1000], 0, True),  # more than 32 ranges: one atomic per request
    (50_000, [3] * 500 + [1_000_003] + [7] * 500, 1, False), (45_001, [100_000] * 9, 2, False), (45_001, [131_072] * 3 + [0] * 70 + [1], 0, False),
    (50_000, [37] * 3000, 0, False), (20_000, [300_000, 5], 3, True), (300, [100] * 400, 1, False),
]


@pytest.mark.parametrize("K,sizes,skip,bad", CASES, ids=[f"{c[0]}_{len(c[1])}" for c in CASES])
def test_count_ranges(K, sizes, skip, bad):
    n, J = sum(sizes), len(sizes)
    rng = np.random.default_rng(K + J)
    keys = np.minimum(rng.geometric(0.001, n) - 1 + rng.integers(0, 2, n) * rng.integers(0, K, n), K - 1)
    keys[:: max(1, n // 50)] = K - 1
    if bad:
        keys = np.where(rng.random(n) < 0.01, K + rng.integers(0, 5, n), keys)
        keys[n // 2] = 0xFFFFFFFF
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    say(f"[case] count K={K} J={J} n={n}")
    buf = torch.empty(n + 8, dtype=torch.int32, device="cuda")
    dev = buf[skip:skip + n]
    dev.copy_(torch.from_numpy(keys.astype(np.uint32).view(np.int32)))
    counts = torch.full((J, K), 7, dtype=torch.int32, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.cr_count_rates(dev, torch.from_numpy(off).cuda(), J, K, counts, err)
    got = counts.cpu().numpy()
    for j in range(J):
        part = keys[off[j]:off[j + 1]]
        np.testing.assert_array_equal(got[j], np.bincount(part[part < K], minlength=K))
    assert int(err) == (B.CR_ERR_KEY_RANGE if bad else 0)
