"""GPU parity of the partition at the edges of its sub-tiles and rows. More than 64
destinations: sub-tiles of 8,192 requests with one interval and 128 of them or more, else of
4,096, 1,024 per wavefront; request counts around whole sub-tiles and wavefronts, padded and full
destination rows, skewed and uniform destinations, few and many blocks. Up to 64: counter rows
of an odd number of 16-byte pieces, under the staged records."""
import numpy as np
import pytest

from oracle import pipeline as opipe
from paper_2608_19677_amd import workload as wl_mod
from paper_2608_19677_amd.pipeline import Pipeline

from cr_check import compare_all, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [65, 257, 1023, 1024])
@pytest.mark.parametrize("n,J,P", [(1, 1, 2), (8192 * 3, 1, 3), (8192 * 5 + 1025, 1, 64), (8192 * 4 + 63, 1, 64), (4096 * 7 + 1030, 1, 4), (4096 * 2, 3, 2),
                                   (4096 * 4 + 1023, 7, 64), (4096 * 5 + 1, 30, 64)])
def test_wide_partition_parity(R, n, J, P):
    wl = wl_mod.small_random(R + n % 89, num_keys=1500, n=n, R=R, Ws=[4 + 3 * (c % 9) for c in range(P)], J=J)
    if J > 1:  # one key for a stretch: whole chunks of one destination
        wl.keys[n // 3: n // 3 + 2500] = wl.keys[0]
    say(f"[case] R={R} n={n} J={J} P={P}")
    gp = Pipeline(wl)
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl))


@pytest.mark.parametrize("R", [1, 8, 9, 16, 57, 63, 64])
@pytest.mark.parametrize("n,J,P", [(1, 1, 1), (1024, 1, 9), (8 * 1024 + 8, 1, 5), (9 * 1024 + 17, 11, 3)])
def test_narrow_partition_parity(R, n, J, P):
    wl = wl_mod.small_random(50 + R + n % 89, num_keys=700, n=n, R=R, Ws=[4 + 3 * (c % 9) for c in range(P)], J=J)
    if J > 1:
        wl.keys[n // 3: n // 3 + 2500] = wl.keys[0]
    say(f"[case] R={R} n={n} J={J} P={P}")
    gp = Pipeline(wl)
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl))
