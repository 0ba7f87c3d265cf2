"""GPU parity of live-load dispatch where its batches change form: member lists of one lane and
of several rounds of 64 lanes, every destination a member, batches with and without replicated
keys in one interval, partial last batches, loads that tie."""
import pytest

from oracle import pipeline as opipe
from paper_2608_19677_amd import workload as wl_mod
from paper_2608_19677_amd.pipeline import Pipeline

from cr_check import compare_all, say

pytestmark = pytest.mark.gpu

CASES = [
    # seed, K, n, R, Ws, J, hot, hot_share, qs
    (51, 200, 9_001, 64, [20], 2, 2, 0.9, [(1, 20)]),        # k clamped to 64 lanes
    (52, 3000, 20_003, 65, [9, 30], 3, 1, 0.9, [(1, 1)]),    # one list just under 64, one destination past a lane
    (53, 3000, 20_003, 200, [9], 2, 2, 0.8, [(1, 1)]),       # lists of two rounds
    (54, 2000, 12_001, 1024, [4], 2, 1, 0.95, [(1, 2)]),     # lists of up to 1,024 members
    (55, 5000, 30_017, 30, [16], 4, 1, 0.01, [(1, 4)]),      # replicated keys in some batches only
    (56, 5000, 30_017, 300, [3], 4, 0, 0.0, [(1, 1)]),
    (57, 5000, 64 * 40 + 1, 2, [40], 1, 0, 0.0, [(3, 2)]),
]


@pytest.mark.parametrize("case", CASES, ids=[f"m{c[0]}" for c in CASES])
def test_live_members(case):
    seed, K, n, R, Ws, J, hot, share, qs = case
    wl = wl_mod.small_random(seed, num_keys=K, n=n, R=R, Ws=Ws, J=J, hot=hot, hot_share=share, qs=qs)
    say(f"[case] live members m{seed} R={R}")
    gp = Pipeline(wl, dispatch="live")
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl, dispatch="live"))


@pytest.mark.parametrize("R", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("W,n,hot", [(1, 64 * 90 + 3, 0), (40, 20_001, 0), (6, 9_000, 2)])
def test_live_few_destinations(R, W, n, hot):
    # both sides of the line between masks as ballots and masks in LDS: hardly anything admitted
    # (many passes per batch), most of it, and batches with replicated keys between the others
    wl = wl_mod.small_random(60 + R, num_keys=1200, n=n, R=R, Ws=[W], J=5, hot=hot, hot_share=0.02 * hot, qs=[(1, 8 if hot else 1)])
    say(f"[case] live, R={R} W={W}")
    gp = Pipeline(wl, dispatch="live")
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl, dispatch="live"))
