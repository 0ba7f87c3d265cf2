"""GPU parity of the plan build at the sizes where its kernels change form: admission budgets
around the two block sizes, key indexes in LDS and (beyond 1,179,648 keys) in global memory,
heads of keys with k > 1 longer than a block or cut inside one, windows admitted whole."""
import numpy as np
import pytest
import torch

import oracle
from oracle import pipeline as opipe
from paper_2608_19677_amd import binding as B
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


# Long runs of equal counts over 65 to 1,024 destinations (LPT by epochs): runs shorter and
# longer than 64 rounds, loads that cross powers of two inside a run, everything admitted
# (loads from zero), whales that stay ahead of the rest, fractional charges.
LPT = [
    # seed, K, n, R, W, J, hot, hot_share, q, zipf
    (311, 30_000, 90_000, 65, 400, 1, 2, 0.2, (1, 1), 0.7),
    (312, 60_000, 150_000, 129, 300, 2, 0, 0.0, (2, 5), 0.3),
    (313, 60_000, 400_000, 257, 256, 1, 5, 0.6, (1, 2), 0.2),
    (314, 200_000, 300_000, 512, 300, 1, 0, 0.0, (1, 1), 0.1),
    (315, 250_000, 900_000, 1024, 256, 1, 3, 0.5, (3, 7), 0.4),
    (316, 70_000, 70_000, 1000, 512, 1, 0, 0.0, (1, 1), 0.0),
    (317, 3000, 300_000, 700, 30, 3, 0, 0.0, (1, 9), 0.05),
    (318, 40_000, 200_000, 30, 512, 2, 2, 0.3, (1, 1), 0.5),
    (319, 40_000, 120_000, 64, 512, 1, 0, 0.0, (2, 3), 0.2),
    (320, 9000, 200_000, 7, 512, 1, 1, 0.4, (1, 2), 0.1),
]


@pytest.mark.parametrize("case", LPT, ids=[f"r{c[3]}_{c[0]}" for c in LPT])
def test_lpt_runs_of_equal_counts(case):
    seed, K, n, R, W, J, hot, share, q, zipf = case
    wl = wl_mod.small_random(seed, num_keys=K, n=n, R=R, Ws=[W], J=J, hot=hot, hot_share=share, qs=[q], zipf_s=zipf)
    say(f"[case] lpt {seed} K={K} R={R} W={W}")
    gp = Pipeline(wl)
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl))


# The window order of long rows. By one block per window: below 73,728 + 1,536 keys per window,
# and for more than 112 windows. By many blocks (budgets from 1,024 slots): thresholds inside the
# exact bins and inside refined ones, ties cut by key, rows with fewer nonzero keys than slots and
# empty ones, odd row lengths, budgets sorted by one block and, above 4,096 slots, by 1 to 3 radix
# passes, of one window and of several.
WIDE = [
    # K, R, W, windows, kind
    (65_535, 64, 16, 3, "zipf"), (65_537, 32, 64, 5, "zipf"), (128_824, 30, 64, 2, "big"), (70_000, 30, 64, 4, "flat"),
    (66_666, 64, 64, 2, "few"), (65_536, 128, 64, 2, "zipf"), (100_003, 64, 300, 40, "big"), (90_000, 100, 100, 1, "huge"),
    (70_000, 200, 200, 2, "flat"), (262_147, 1024, 128, 1, "zipf"), (66_001, 33, 125, 2, "huge"), (80_001, 64, 65, 1, "one"),
    (200_000, 7, 100, 2, "big"),
    (75_263, 32, 64, 1, "zipf"), (75_264, 32, 64, 1, "zipf"), (76_801, 32, 32, 2, "flat"), (80_003, 64, 64, 4, "flat"), (81_411, 200, 200, 5, "flat"),
    (80_001, 64, 64, 3, "few"), (80_002, 128, 64, 3, "few"), (245_761, 64, 16, 112, "few"), (247_301, 64, 16, 113, "few"),
    (83_003, 64, 300, 3, "mid"), (84_001, 50, 100, 3, "huge"), (90_001, 65, 64, 10, "big"), (79_001, 80, 100, 3, "one"),
]


@pytest.mark.parametrize("K,R,W,NW,kind", WIDE, ids=[f"{c[4]}_{c[0]}_{c[1] * c[2]}" for c in WIDE])
def test_window_order_of_wide_rows(K, R, W, NW, kind):
    rng = np.random.default_rng(K + R)
    if kind == "zipf":
        rows = rng.poisson(3000.0 * (1 + rng.permutation(K)) ** -0.7, (NW, K))
    elif kind == "big":      # thresholds in the thousands: one or two refinements
        rows = rng.integers(2000, 90_000, (NW, K))
    elif kind == "huge":     # up to 2^32 - 1: all three
        rows = rng.integers(1, 1 << 32, (NW, K))
    elif kind == "mid":      # counts of 11 bits
        rows = rng.integers(1, 2000, (NW, K))
    elif kind == "flat":     # ties everywhere
        rows = rng.integers(5, 8, (NW, K))
    elif kind == "few":      # fewer nonzero keys than slots, an empty row
        rows = np.where(rng.random((NW, K)) < 0.02, rng.integers(1, 500, (NW, K)), 0)
        rows[-1] = 0
    else:                    # one value
        rows = np.full((NW, K), 70_001)
    rows = rows.astype(np.uint32)
    say(f"[case] wide rows {kind} K={K} Cmax={R * W}")
    specs = [(w, W, B.CR_WINDOW_SUM, 1, 1, B.CR_PLAN_AFFINITY, 0) for w in range(NW)]
    ps = B.PlanSet(specs, 1, R, W, K, NW, "cuda")
    ws = torch.empty(B.cr_admit_workspace_bytes(NW, R, W), dtype=torch.uint8, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.cr_admit(torch.from_numpy(rows.view(np.int32)).cuda(), ps.c, ws, err)
    torch.cuda.synchronize()
    for w in range(NW):
        keys = np.nonzero(rows[w])[0]
        keys = keys[np.lexsort((keys, -rows[w][keys].astype(np.int64)))][: R * W]
        m = int(ps.n_order[w])
        assert m == len(keys) == int(ps.num_admitted[w])
        np.testing.assert_array_equal(ps.order[w, :m].cpu().numpy().view(np.uint32), keys)
        np.testing.assert_array_equal(ps.order_count[w, :m].cpu().numpy().view(np.uint32), rows[w][keys])
        assert int(ps.cold[w]) == int(rows[w].astype(np.uint64).sum() - rows[w][keys].astype(np.uint64).sum())
    assert int(err) == 0


@pytest.mark.parametrize("R,W", [(64, 16), (43, 32), (32, 64), (64, 64), (50, 100)])
def test_wide_rows_leave_unused_entries_alone(R, W):
    # entries of order and order_count past n_order are the caller's; rows of few nonzero keys, of
    # counts wide enough for every refinement (kept whole rows), and an empty one
    K, NW = 80_009, 3
    rng = np.random.default_rng(R)
    rows = np.zeros((NW, K), np.uint32)
    rows[0, rng.choice(K, 700, replace=False)] = rng.integers(1, 1 << 32, 700)
    rows[1] = rng.integers(1, 1 << 32, K)
    say(f"[case] unused entries, Cmax={R * W}")
    ps = B.PlanSet([(w, W, B.CR_WINDOW_SUM, 1, 1, B.CR_PLAN_AFFINITY, 0) for w in range(NW)], 1, R, W, K, NW, "cuda")
    ps.order.fill_(0x5A5A5A5A)
    ps.order_count.fill_(0x3C3C3C3C)
    ws = torch.empty(B.cr_admit_workspace_bytes(NW, R, W), dtype=torch.uint8, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.cr_admit(torch.from_numpy(rows.view(np.int32)).cuda(), ps.c, ws, err)
    assert int(err) == 0
    for w, m in enumerate((700, R * W, 0)):
        keys = np.nonzero(rows[w])[0]
        keys = keys[np.lexsort((keys, -rows[w][keys].astype(np.int64)))][:m]
        got, cnt = ps.order[w].cpu().numpy(), ps.order_count[w].cpu().numpy()
        assert int(ps.n_order[w]) == m
        np.testing.assert_array_equal(got[:m].view(np.uint32), keys)
        np.testing.assert_array_equal(cnt[:m].view(np.uint32), rows[w][keys])
        assert np.all(got[m:] == 0x5A5A5A5A) and np.all(cnt[m:] == 0x3C3C3C3C)


@pytest.mark.parametrize("R", [64, 65, 300])
def test_lpt_loads_beyond_the_integers_of_a_double(R):
    # equal counts on loads of 2^53 and more: every charge rounds, so no two may be added as one
    K = int(R * 2**53 / (2**32 - 1) * 1.01) // 64 * 64 + 3
    W = 5 * 1024 // R
    say(f"[case] loads past 2^53, R={R} K={K}")
    counts = torch.full((1, K), -1, dtype=torch.int32, device="cuda")
    ps = B.PlanSet([(0, W, B.CR_WINDOW_SUM, 1, 1, B.CR_PLAN_FULL, 0)], 1, R, W, K, 1, "cuda")
    ws = torch.empty(B.cr_admit_workspace_bytes(1, R, W), dtype=torch.uint8, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.cr_admit(counts, ps.c, ws, err)
    B.cr_place_lpt(counts, ps.c)
    A = R * W
    cold = (K - A) * (2**32 - 1)
    members, _, load = oracle.place_lpt(np.arange(A, dtype=np.uint32), np.ones(A, np.uint32), np.full(A, 0xFFFFFFFF, np.uint32), R, cold)
    assert int(err) == 0 and int(ps.num_admitted[0]) == A and int(ps.cold[0]) == cold and load.min() >= 2.0**53
    np.testing.assert_array_equal(ps.members[0, :A].cpu().numpy().view(np.uint16), members)
    np.testing.assert_array_equal(ps.load[0].cpu().numpy().view(np.uint64), load.view(np.uint64))


@pytest.mark.parametrize("R", [65, 128, 129, 256, 257, 512, 513, 1024])
@pytest.mark.parametrize("kind", ["distinct", "steps", "pairs", "ties"])
def test_lpt_batches_of_few_and_many_counts(R, kind):
    # batches of one to many counts, in order or not (merged by runs, or sorted), runs of one
    # count around the lengths from which they are placed by epochs, k > 1 in front
    rng = np.random.default_rng(R)
    W = 12
    A = R * W
    if kind == "distinct":
        c = 50_000 + np.arange(A)[::-1] * rng.integers(1, 4)
    elif kind == "steps":    # runs of 1 to 7 R jobs, steps small and large
        c = np.repeat(np.cumsum(rng.integers(1, 900, 64))[::-1] + 40_000, rng.integers(1, 7 * R, 64))[:A]
    elif kind == "pairs":    # two or three counts per batch
        c = np.repeat(np.cumsum(rng.integers(1, 300, A))[::-1] + 5000, rng.integers(R // 3 + 1, R, A))[:A]
    else:                    # loads that meet
        c = np.sort(rng.choice([1, 2, 4, 8, 64, 3000], A, p=[0.3, 0.2, 0.2, 0.2, 0.09, 0.01]))[::-1]
    K = A + 50
    row = np.zeros(K, np.uint32)
    row[: len(c)] = c
    row[len(c):] = 1
    say(f"[case] lpt batches {kind} R={R}")
    counts = torch.from_numpy(row.view(np.int32)).cuda()[None].contiguous()
    ps = B.PlanSet([(0, W, B.CR_WINDOW_SUM, 1, 1, B.CR_PLAN_FULL, 0)], 1, R, W, K, 1, "cuda")
    ws = torch.empty(B.cr_admit_workspace_bytes(1, R, W), dtype=torch.uint8, device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.cr_admit(counts, ps.c, ws, err)
    B.cr_place_lpt(counts, ps.c)
    assert int(err) == 0
    a = int(ps.num_admitted[0])
    off = ps.member_off[0, : a + 1].cpu().numpy()
    keys = ps.order[0, :a].cpu().numpy().astype(np.uint32)
    members, _, load = oracle.place_lpt(keys, np.diff(off).astype(np.uint32), row, R, int(ps.cold[0]))
    np.testing.assert_array_equal(ps.members[0, : off[-1]].cpu().numpy().view(np.uint16), members)
    np.testing.assert_array_equal(ps.load[0].cpu().numpy().view(np.uint64), load.view(np.uint64))
