"""GPU parity of the replay of caches of 64 slots and more (a hash table and position bitmap
per wavefront, 64 records per step) where its bookkeeping turns over: slot budgets at both
ends of every table size, streams of one hot set (the bitmap runs full without a miss),
streams that never repeat a key (the table runs full), keys repeated inside one step, out-of-range
keys and carried cache state; and, in streams of more records than a segment's rebuild may scan
(64 segments or 65,536 records), stretches of fewer keys than slots, whose segments the
sequential pass replays."""
import numpy as np
import pytest

from oracle import pipeline as opipe
from paper_2608_19677_amd import binding as B
from paper_2608_19677_amd import workload as wl_mod
from paper_2608_19677_amd.pipeline import Pipeline

from cr_check import compare_all, say

pytestmark = pytest.mark.gpu

EDGES = [64, 65, 96, 97, 192, 193, 384, 385, 511, 512]


def _stream(kind, n, K, rng):
    if kind == "cycle":      # one key more than a cache holds, round robin: every access misses
        return np.arange(n) % K
    if kind == "distinct":   # no key comes back
        return rng.permutation(np.arange(n) % K)
    if kind == "hot":        # few keys, all hits after the first
        return rng.integers(0, min(K, 40), n)
    if kind == "runs":       # every key several times in a row
        return np.repeat(rng.integers(0, K, n // 5 + 1), 5)[:n]
    p = 1.0 / np.arange(1, K + 1) ** 0.9
    return rng.choice(K, n, p=p / p.sum())


@pytest.mark.parametrize("kind,K,R,J", [("zipf", 5000, 3, 1), ("zipf", 900, 2, 40), ("cycle", 513, 1, 3), ("cycle", 193, 1, 1),
                                        ("distinct", 30_000, 1, 2), ("hot", 1000, 2, 5), ("runs", 3000, 2, 7)])
def test_hash_replay_parity(kind, K, R, J):
    n = 30_011
    rng = np.random.default_rng(K + J)
    wl = wl_mod.small_random(900 + K % 97, num_keys=K, n=n, R=R, Ws=EDGES, J=J)
    wl.keys = _stream(kind, n, K, rng).astype(np.uint32)
    say(f"[case] {kind} K={K} R={R} J={J}")
    gp = Pipeline(wl)
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl))


def test_hash_replay_out_of_range_keys_and_carried_state():
    """Two chunks, the second from the first's caches, with keys past num_keys in both:
    skipped, flagged, and without effect on the caches."""
    K, R, n = 2500, 2, 20_500
    wl = wl_mod.small_random(77, num_keys=K, n=n, R=R, Ws=EDGES, J=1)
    bad = np.random.default_rng(5).random(n) < 0.03
    wl.keys = np.where(bad, K + 7, wl.keys).astype(np.uint32)
    say("[case] out-of-range keys, carried state")
    first = Pipeline(wl)
    first.step()
    second = Pipeline(wl, lru_in=first.lru_out)
    second.step()
    o1 = opipe.run(wl)
    o2 = opipe.run(wl, lru=o1["lru"])
    for gp, o in ((first, o1), (second, o2)):
        h = gp.host()
        assert h["err"] == B.CR_ERR_KEY_RANGE
        np.testing.assert_array_equal(h["stats"], o["stats"])
        for c, cand in enumerate(wl.candidates):
            np.testing.assert_array_equal(h["lru"][c, :, : cand.W], o["lru"][c])


def _stretches(n, cuts, K, few, rng):
    """Zipf keys, then `few` keys only from cuts[0] to cuts[1], then Zipf keys again."""
    keys = _stream("zipf", n, K, rng)
    keys[cuts[0]:cuts[1]] = rng.integers(0, few, cuts[1] - cuts[0]) * 3 + 1
    return keys.astype(np.uint32)


@pytest.mark.parametrize("few,J", [(1, 1), (40, 4), (63, 1), (300, 9)])
def test_hash_replay_segments_out_of_rebuild_budget(few, J):
    # 640,000 records of few keys over one destination: more than any of the budgets reaches back
    # (524,288 records at 512 slots); with 300 keys the budgets up to 193 slots are not marked
    n = 760_003
    rng = np.random.default_rng(few)
    wl = wl_mod.small_random(400 + few, num_keys=5000, n=n, R=1, Ws=EDGES, J=J)
    wl.keys = _stretches(n, (50_000, 690_000), 5000, few, rng)
    say(f"[case] out of budget, {few} keys J={J}")
    gp = Pipeline(wl)
    gp.step()
    compare_all(wl, gp, gp.host(), opipe.run(wl, threads=8))


def test_hash_replay_out_of_budget_from_carried_state_with_bad_keys():
    # a stream of few keys from its first record on, so that the marked segments' rebuild ends
    # with the caches of the chunk before; keys past num_keys in both chunks
    K, n = 3000, 600_007
    rng = np.random.default_rng(8)
    wl = wl_mod.small_random(78, num_keys=K, n=n, R=1, Ws=EDGES, J=1)
    wl.keys = _stretches(n, (0, 590_000), K, 50, rng)
    wl.keys[rng.random(n) < 0.02] = K + 9
    head = wl_mod.small_random(79, num_keys=K, n=40_000, R=1, Ws=EDGES, J=1)
    head.keys = np.where(rng.random(40_000) < 0.05, K + 1, _stream("zipf", 40_000, K, rng)).astype(np.uint32)
    say("[case] out of budget, carried state, out-of-range keys")
    first = Pipeline(head)
    first.step()
    o1 = opipe.run(head)
    second = Pipeline(wl, lru_in=first.lru_out)
    second.step()
    o2 = opipe.run(wl, lru=o1["lru"], threads=8)
    h = second.host()
    assert h["err"] == B.CR_ERR_KEY_RANGE
    np.testing.assert_array_equal(h["stats"], o2["stats"])
    for c, cand in enumerate(wl.candidates):
        np.testing.assert_array_equal(h["lru"][c, :, : cand.W], o2["lru"][c])
