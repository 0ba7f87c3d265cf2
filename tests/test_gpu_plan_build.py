"""GPU parity of the plan build at the sizes where its kernels change form: admission budgets
around the two block sizes, key indexes in LDS and (beyond 1,179,648 keys) in global memory,
heads of keys with k > 1 longer than a block or cut inside one, windows admitted whole."""
import numpy as np
import pytest

from oracle import pipeline as opipe
from paper_2608_19677_amd import workload as wl_mod
from paper_2608_19677_amd.pipeline import Pipeline

from cr_check import compare_all, say

pytestmark = pytest.mark.gpu

ADMIT = [
    # seed, K, n, R, Ws, J, hot, hot_share, qs, zipf
    (301, 1_200_000, 60_000, 5, [9], 2, 2, 0.3, [(1, 1)], 0.6),       # key index in global memory
    (302, 9000, 200_000, 128, [64, 65], 1, 0, 0.0, [(1, 50)], 0.5),   # Cmax 8,192 and above; every key k > 1
    (303, 9000, 200_000, 127, [64, 200], 3, 5, 0.4, [(1, 1), (1, 400)], 0.9),  # budget ends inside the head
    (304, 3000, 90_000, 30, [4, 90], 2, 0, 0.0, [(1, 4), (2, 5)], 1.5),        # k clamped to R, few keys fit
    (305, 40, 5_000, 64, [2, 512], 1, 0, 0.0, [(1, 1)], 1.0),         # every key admitted
]


@pytest.mark.parametrize("case", ADMIT, ids=[f"p{c[0]}" for c in ADMIT])
def test_admission_edges(case):
    seed, K, n, R, Ws, J, hot, share, qs, zipf = case
    wl = wl_mod.small_random(seed, num_keys=K, n=n, R=R, Ws=Ws, J=J, hot=hot, hot_share=share, qs=qs, zipf_s=zipf)
    say(f"[case] p{seed} K={K} R={R} Ws={Ws} qs={qs}")
    gp = Pipeline(wl)
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl))
