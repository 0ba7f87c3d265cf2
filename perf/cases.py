"""Performance cases: the work users have this framework do, through its public entry points.

Kinds of case (``kind``):

* ``step``   one ``Pipeline.step()``: count, admission, placement, dispatch, partition and
             LRU replay of a request stream, launched eagerly or (``graph``) replayed as the
             step captured once as a HIP graph;
* ``drift``  the same step for the replanning study (plan windows named per interval,
             statistics in finer bins), followed by the churn of the plans;
* ``live``   live-load dispatch of a stream through plans already built;
* ``plan``   admission and placement from counts already in hand;
* ``remap``  opaque 32-bit ids: directory build, lookup of the stream and scatter of the
             per-key prefix lengths.

Inputs are drawn on the GPU from the seed alone. Sizes are those of the named workloads
(``paper_2608_19677_amd/workload.py``), of the tests, or generic ones in between.
"""
from __future__ import annotations

import heapq
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2608_19677_amd import binding as B
from paper_2608_19677_amd.keymap import KeyMap
from paper_2608_19677_amd.pipeline import DeviceInputs, Pipeline
from paper_2608_19677_amd.workload import SWEEP_W, Candidate, water_fill, zipf_probs

DEV = "cuda"

SWEEP_WS = ",".join(str(w) for w in SWEEP_W)
SWEEP_QS = ",".join(f"{28 + 2 * m}/35" for m in range(8))


def _case(name, kind, **kw):
    """A case with the defaults of a plain one-plan step."""
    c = dict(kind=kind, n=0, K=1000, R=30, W="64", q="1/1", variants="full", J=1, cuts="even", cv=1.0, zipf=1.0, cap=0.0,
             hot=0, hot_share=0.0, sigma=0.0, bins=0, chunk=False, graph=False)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: one interval of 1,000 keys over 30 caches, launched eagerly (unit
        # tests, notebooks, a first look at a log): launch count and host path.
        _case("tiny_eager", "step", n=100_000, K=1000, R=30, W="16", zipf=1.1),
        # A short ragged log with two slot budgets: odd sizes, destinations just past one
        # wavefront, uneven intervals.
        _case("small_ragged", "step", n=77_777, K=2003, R=65, W="63,130", J=9, cuts="ragged", zipf=1.1, hot=3, hot_share=0.2),
        # The 70B-like day: 1e7 requests, a plan per 60-second interval, as the captured step.
        _case("llama70b_graph", "step", n=10_000_000, K=20_000, R=30, W="64", J=948, cap=0.003, graph=True),
        # The component ablation: four plan variants over the injected-whale stream.
        _case("ablation_step", "step", n=20_000_000, K=5008, R=16, W="128", q="2/5", variants="flat,affinity,replicated,full", J=667, zipf=1.1, hot=8, hot_share=0.48),
        # The burst stream: 50,000 keys, 100 intervals of about half a million requests.
        _case("burst_step", "step", n=50_000_000, K=50_000, R=64, W="64", J=100, cv=30.0, zipf=1.2),
        # The replanning study: six candidates by plan window, 600 statistics bins, churn.
        _case("drift_study", "drift", n=6_000_000, K=20_000, R=30, W="64", J=6, cap=0.003, sigma=0.3, bins=600),
        # Live-load dispatch of the 70B-like stream with bursty (Gamma, CV 1.9) arrivals.
        _case("live_gamma", "live", n=10_000_000, K=20_000, R=30, W="64", J=948, cv=1.9, cap=0.003),
        # A log that arrives with salted ids: remapped to dense keys before anything else.
        _case("opaque_remap", "remap", n=10_000_000, K=20_000),
        # A log of some millions of requests over more keys than a CU's LDS counts, several
        # hours, four candidate plans, odd everything.
        _case("ragged_mid", "step", n=4_000_037, K=128_824, R=257, W="26,156", q="1/1,2/5", J=24, cuts="ragged", zipf=0.9),
        # One periodic plan build at the size the paper times (128,824 keys, 30 replicas).
        _case("plan_paper", "plan", n=20_000_000, K=128_824, R=30, W="64", zipf=0.9),
        # One plan build for a large fleet (1,000,000 keys, 1,024 replicas, 512 slots each).
        _case("plan_large", "plan", n=100_000_000, K=1_000_000, R=1024, W="512", q="34/35", zipf=0.9),
        # The large sweep: one 1e8-request chunk under 64 candidate plans, planned from the
        # chunk before it, caches carried over.
        _case("sweep_chunk", "step", n=100_000_000, K=1_000_000, R=1024, W=SWEEP_WS, q=SWEEP_QS, zipf=0.9, chunk=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["drift", "live", "plan", "plan", "remap"])
    zipf = round(rng.uniform(0.8, 1.25), 3)
    hot = rng.choice([0, 0, rng.randint(1, 8)])
    mix = dict(zipf=zipf, hot=hot, hot_share=round(rng.uniform(0.05, 0.5), 3) if hot else 0.0)
    if kind == "remap":
        n = _log(rng, 20_000, 40_000_000)
        return _case(None, kind, n=n, K=min(n, _log(rng, 500, 2_000_000)), **mix)
    K = _log(rng, 500, 1_000_000)
    R = rng.choice([rng.randint(2, 64), rng.choice([8, 16, 30, 32, 64]), rng.randint(65, 1024)])
    q = lambda: f"{rng.randint(8, 42)}/{35}"  # noqa: E731
    if kind == "plan":
        J = rng.choice([1, 1, rng.randint(2, 64)])
        while J * K > 20_000_000:
            J = J // 2
        n = _log(rng, 20_000, 100_000_000)
        return _case(None, kind, n=n, K=K, R=R, W=str(_log(rng, 4, 512)), q=q(), J=max(J, 1), **mix)
    if kind == "live":
        n = _log(rng, 20_000, 20_000_000)
        J = max(n // _log(rng, 2000, 20_000), 1)
        K = min(K, max(500, 40_000_000 // J))
        R = min(R, 128) if J > 100 else R
        W = min(_log(rng, 4, 256), max(4, 60_000_000 // (J * R)))
        return _case(None, kind, n=n, K=K, R=R, W=str(W), q=q(), J=min(J, 2000), cv=round(rng.uniform(0.5, 3.0), 2), **mix)
    if kind == "drift":
        n = _log(rng, 100_000, 6_000_000)
        J = rng.randint(2, 6)
        return _case(None, kind, n=n, K=min(K, 100_000), R=min(R, 256), W=str(_log(rng, 8, 128)), J=J, sigma=0.3,
                     bins=J * rng.randint(1, 100), **mix)
    shape = rng.choice(["one", "few", "many", "sweep", "ablation"])
    n = _log(rng, 10_000, 50_000_000)
    if shape == "sweep":  # many candidates of one window
        n = _log(rng, 50_000, 20_000_000)
        P = rng.choice([8, 9, 16, 24, 32])
        nw = rng.choice([1, 2, 4]) if P % 4 == 0 else 1
        ws = sorted(_log(rng, 4, 512) for _ in range(nw))
        qs = sorted(q() for _ in range(P // nw))
        return _case(None, "step", n=n, K=K, R=R, W=",".join(map(str, ws)), q=",".join(qs), chunk=True, **mix)
    if shape == "ablation":
        n = _log(rng, 20_000, 20_000_000)
        J = min(_log(rng, 1, 400), max(1, n // 500))
        K = min(K, max(500, 40_000_000 // J))
        R = min(R, 64)
        W = min(_log(rng, 8, 256), max(8, 40_000_000 // (4 * J * R)))
        return _case(None, "step", n=n, K=K, R=R, W=str(W), q=q(), variants="flat,affinity,replicated,full", J=J, **mix)
    J = 1 if shape == "one" else (rng.randint(2, 30) if shape == "few" else min(_log(rng, 30, 1000), max(2, n // 500)))
    K = min(K, max(500, 40_000_000 // J))
    nw = rng.choice([1, 1, 2, 3])
    ws = sorted(min(_log(rng, 4, 512), max(4, 60_000_000 // (nw * J * R))) for _ in range(nw))
    return _case(None, "step", n=n, K=K, R=R, W=",".join(map(str, ws)), q=q(), J=J, cuts=rng.choice(["even", "ragged"]),
                 graph=shape == "many" and rng.random() < 0.5, **mix)


# -- inputs -------------------------------------------------------------------------------
def _candidates(case):
    ws = [int(x) for x in case["W"].split(",")]
    qs = [tuple(int(v) for v in x.split("/")) for x in case["q"].split(",")]
    vs = case["variants"].split(",")
    out = [Candidate(w, a, b, v, 7 if v in ("affinity", "replicated") else 0) for w in ws for a, b in qs for v in vs]
    return [out[0]] * case["J"] if case["kind"] == "drift" else out


def _offsets(case, seed):
    """Interval starts: `even` intervals of about n / J requests (arrivals of coefficient of
    variation cv), or `ragged` ones cut anywhere."""
    n, J = case["n"], case["J"]
    rng = np.random.Generator(np.random.PCG64([seed, 11]))
    if case["kind"] == "drift":
        inner = np.arange(1, J) * (n // J)
    elif case["cuts"] == "ragged":
        inner = np.sort(rng.integers(0, n + 1, size=J - 1))
    else:
        m = n / J
        inner = np.minimum(n, np.cumsum(np.rint(np.maximum(0.0, rng.normal(m, case["cv"] * math.sqrt(m), size=J - 1)))))
    return np.concatenate([[0], inner, [n]]).astype(np.uint64)


def _probs(case):
    p = zipf_probs(case["K"], case["zipf"])
    if case["cap"]:
        p = water_fill(p, max(case["cap"], 1.01 / case["K"]))
    if case["hot"]:
        h = min(case["hot"], case["K"])
        p = p * (1.0 - case["hot_share"])
        p[:h] += case["hot_share"] / h
    return p / p.sum()


def _gen(seed, tag):
    return torch.Generator(device=DEV).manual_seed(seed * 1000 + tag)


def _sample(p, perm, n, gen, out=None):
    """n keys drawn from p by rank, through the permutation (int32 on the GPU)."""
    cdf = torch.cumsum(p, 0)
    out = torch.empty(n, dtype=torch.int32, device=DEV) if out is None else out
    for s in range(0, n, 1 << 25):
        e = min(n, s + (1 << 25))
        u = torch.rand(e - s, dtype=torch.float64, device=DEV, generator=gen) * cdf[-1]
        r = torch.searchsorted(cdf, u, right=True).clamp_(max=p.numel() - 1)
        out[s:e] = perm[r]
    return out


def _stream(case, seed, off):
    p = torch.from_numpy(_probs(case)).to(DEV)
    K, n = case["K"], case["n"]
    perm = torch.randperm(K, device=DEV, generator=_gen(seed, 1)).to(torch.int32)
    gen = _gen(seed, 2)
    if not case["sigma"]:
        return _sample(p, perm, n, gen), p, perm
    keys = torch.empty(n, dtype=torch.int32, device=DEV)  # lognormal random walk of the shares per interval
    walk, w = _gen(seed, 3), p
    for j in range(case["J"]):
        if j:
            w = w * torch.exp(case["sigma"] * torch.randn(K, dtype=torch.float64, device=DEV, generator=walk))
        a, b = int(off[j]), int(off[j + 1])
        _sample(w / w.sum(), perm, b - a, gen, keys[a:b])
    return keys, p, perm


def _prefix_lengths(K, seed):
    z = torch.randn(K, device=DEV, generator=_gen(seed, 4))
    return torch.clamp(torch.round(2000.0 * torch.exp(0.5 * z)), min=1.0).to(torch.int32)


def _counts(keys, K):
    return torch.bincount(keys, minlength=K).to(torch.int32)


def _carried(case, cands, seed):
    """Full caches: W distinct keys per candidate and destination, as an earlier chunk left them."""
    K, R, P = case["K"], case["R"], len(cands)
    mw = max(c.W for c in cands)
    step = 7919 % K or 1
    while math.gcd(step, K) != 1:
        step += 1
    base = torch.randint(0, K, (P, R, 1), device=DEV, generator=_gen(seed, 5))
    slot = torch.arange(mw, device=DEV)
    keys = ((base + slot * step) % K).to(torch.int32)
    used = torch.tensor([min(c.W, K) for c in cands], device=DEV).view(P, 1, 1)
    return torch.where(slot < used, keys, torch.full_like(keys, -1))


def _zero_plans(ps):
    """Entries a plan does not use are never written: give them a value."""
    for t in (ps.order, ps.order_count, ps.member_off, ps.members, ps.route):
        t.zero_()


def prepare(case, seed):
    K, R, n = case["K"], case["R"], case["n"]
    off = _offsets(case, seed)
    if case["kind"] == "remap":
        keys, _, _ = _stream(case, seed, off)
        salt = seed % 0xFFFF
        ids_of = ((torch.arange(K, device=DEV) * 0x9E3779B1 + salt) & 0xFFFFFFFF) ^ (salt << 8)
        ids_of = torch.where(ids_of == 0xFFFFFFFF, torch.zeros_like(ids_of), ids_of)
        ids_of = torch.where(ids_of >= 1 << 31, ids_of - (1 << 32), ids_of).to(torch.int32)
        km = KeyMap(K, DEV)
        return SimpleNamespace(case=case, km=km, ids=ids_of[keys.long()], attr=ids_of, plen=_prefix_lengths(K, seed),
                               dense=torch.empty(n, dtype=torch.int32, device=DEV), out=torch.zeros(K, dtype=torch.int32, device=DEV),
                               err=torch.zeros(1, dtype=torch.int32, device=DEV))
    cands = _candidates(case)
    J, P = case["J"], len(cands)
    if case["kind"] == "plan":
        p = torch.from_numpy(_probs(case)).to(DEV)
        counts = torch.empty((J, K), dtype=torch.int32, device=DEV)
        for j in range(J):
            perm = torch.randperm(K, device=DEV, generator=_gen(seed, 20 + j)).to(torch.int32)
            counts[j] = _counts(_sample(p, perm, max(n // J, 1), _gen(seed, 20_000 + j)), K)
        specs = [(j, c.W, B.CR_WINDOW_SUM, c.a, c.b, B.PLAN_VARIANTS[c.variant], c.place_seed) for j in range(J) for c in cands]
        ps = B.PlanSet(specs, P, R, max(c.W for c in cands), K, J, DEV)
        _zero_plans(ps)
        ws = torch.empty(B.cr_admit_workspace_bytes(J, R, ps.max_W), dtype=torch.uint8, device=DEV)
        return SimpleNamespace(case=case, counts=counts, ps=ps, ws=ws, err=torch.zeros(1, dtype=torch.int32, device=DEV))
    keys, p, perm = _stream(case, seed, off)
    suffix = torch.randint(50, 401, (n,), dtype=torch.int16, device=DEV, generator=_gen(seed, 6))
    wl = SimpleNamespace(num_keys=K, R=R, candidates=cands, J=J, P=P, n=n, seed=seed, first_index=0, plan_windows=None, stat_offsets=None)
    if case["kind"] == "drift":
        pw = np.tile(np.arange(J)[:, None], (1, J))
        for t in range(1, J):
            pw[t, t] = t - 1
        wl.plan_windows = pw
        wl.stat_offsets = np.rint(np.linspace(0, n, case["bins"] + 1)).astype(np.uint64)
    inp = DeviceInputs(keys=keys, suffix=suffix, prefix_len=_prefix_lengths(K, seed), off=torch.from_numpy(off.view(np.int64)).to(DEV), off_host=off)
    prev = _counts(_sample(p, perm, n, _gen(seed, 7)), K) if case["chunk"] else None
    lru_in = _carried(case, cands, seed) if case["chunk"] else None
    pipe = Pipeline(wl, DEV, dev_in=inp, prev_counts=prev, lru_in=lru_in, dispatch="live" if case["kind"] == "live" else "static")
    _zero_plans(pipe.plans)
    if case["kind"] == "drift":
        pipe.set_churn_pairs([(t * P, t * P + t) for t in range(1, J)] + [((t - 1) * P, t * P) for t in range(1, J)])
    if case["kind"] == "live":
        pipe.count()
        pipe.plan()
    if case["graph"]:
        pipe.capture()
    return SimpleNamespace(case=case, pipe=pipe, err=pipe.err)


def _plan_outputs(ps):
    return dict(order=ps.order, order_count=ps.order_count, n_order=ps.n_order, num_admitted=ps.num_admitted, cold=ps.cold,
                clamped=ps.clamped, member_off=ps.member_off, members=ps.members, load=ps.load, key_index=ps.key_index, route=ps.route)


def run(state):
    kind = state.case["kind"]
    if kind == "remap":
        state.km.build(state.ids, state.err)
        state.km.lookup(state.ids, state.dense)
        state.km.scatter(state.attr, state.plen, state.out)
        return dict(num_keys=state.km.num_keys, dense=state.dense, prefix_len=state.out, err=state.err)
    if kind == "plan":
        B.cr_admit(state.counts, state.ps.c, state.ws, state.err)
        B.cr_place_lpt(state.counts, state.ps.c)
        return dict(_plan_outputs(state.ps), err=state.err)
    p = state.pipe
    if kind == "live":
        p.route()
        return dict(dest=p.dest, err=p.err)
    if state.case["graph"]:
        p.replay_graph()
    else:
        p.step()
    out = dict(_plan_outputs(p.plans), counts=p.counts, dest=p.dest, stats=p.stats, lru=p.lru_out, err=p.err)
    if kind == "drift":
        p.churn()
        out["churn"] = p.churn_out
    return out


# -- what a pass cannot do without ----------------------------------------------------------
def work(case):
    """Inputs read once and outputs written once: 4 B per key, 2 B per suffix, 2 B per
    destination, the counts, the used part of every plan, the statistics and caches; one
    operation per request and plan for each decision (dispatch, cache)."""
    n, K, R, J = case["n"], case["K"], case["R"], case["J"]
    if case["kind"] == "remap":
        return dict(bytes=8.0 * n + 12.0 * K, flops=2.0 * n)
    cands = _candidates(case)
    P = len(cands)
    if case["kind"] == "live":
        return dict(bytes=n * (4.0 + 2.0 * P), flops=float(n * P))
    NW = J if case["kind"] in ("plan", "drift") or case["chunk"] else max(J - 1, 1)
    jobs = sum(0 if c.variant == "flat" else min(K, R * c.W) for c in cands)
    plans = NW * (min(K, R * max(c.W for c in cands)) * 8.0 + jobs * 10.0 + P * (R * 8.0 + (K + 63) // 64 * 16.0))
    if case["kind"] == "plan":
        return dict(bytes=J * K * 4.0 + plans, flops=float(NW * jobs))
    JS = case["bins"] or J
    slots = sum(c.W for c in cands) * R * 4.0
    return dict(bytes=n * (6.0 + 2.0 * P) + K * 4.0 + J * K * 4.0 + plans + JS * P * R * 32.0 + slots * (2 if case["chunk"] else 1),
                flops=2.0 * n * P + NW * jobs)


def tolerance(case):
    # counts, tables, destinations, statistics and caches are whole numbers; the planned loads
    # are doubles added in a fixed order with one rounding per operation
    return "exact"


# -- the planned loads in plain numpy --------------------------------------------------------
def _loads(counts, cand, R):
    """Loads of one plan from one window's counts: Eq. 1, prefix admission, placement."""
    keys = np.nonzero(counts)[0]
    keys = keys[np.lexsort((keys, -counts[keys].astype(np.int64)))]
    c = counts[keys].astype(np.int64)
    N = int(counts.sum())
    if cand.variant == "flat" or N == 0:
        return np.full(R, N / R)
    k = np.ones(len(c), dtype=np.int64) if cand.variant == "affinity" else np.clip(-(-(c * cand.b * R) // (cand.a * N)), 1, R)
    A = int(np.searchsorted(np.cumsum(k), R * cand.W, side="right"))
    L0 = (N - int(c[:A].sum())) / R
    if cand.variant in ("affinity", "replicated"):
        L = np.full(R, L0)
        m32 = lambda x: x & 0xFFFFFFFF  # noqa: E731

        def fmix(x):
            x = m32((x ^ (x >> 16)) * 0x85EBCA6B)
            x = m32((x ^ (x >> 13)) * 0xC2B2AE35)
            return x ^ (x >> 16)
        t = fmix(cand.place_seed ^ 0x7F4A7C15)
        for a in range(A):
            u = fmix(np.int64(fmix(int(keys[a]) ^ t)) ^ np.arange(R, dtype=np.int64))
            for r in np.argsort(u, kind="stable")[: k[a]]:
                L[r] += float(c[a]) / float(k[a])
        return L
    heap = [(L0, r) for r in range(R)]
    for cnt, kk in zip(c[:A].tolist(), k[:A].tolist()):
        if kk == 1:
            v, r = heap[0]
            heapq.heapreplace(heap, (v + cnt, r))
        else:
            for v, r in [heapq.heappop(heap) for _ in range(kk)]:
                heapq.heappush(heap, (v + cnt / kk, r))
    L = np.empty(R)
    for v, r in heap:
        L[r] = v
    return L


def exact(case, seed):
    if case["kind"] in ("remap", "live"):
        return None
    cands = _candidates(case)
    J, K, R = case["J"], case["K"], case["R"]
    jobs = sum({"flat": 0, "full": 1}.get(c.variant, 25) * min(K, R * c.W) for c in cands)
    if J * jobs > 6_000_000 or J * K > 40_000_000:
        return None
    state = prepare(dict(case, graph=False), seed)
    if case["kind"] == "plan":
        rows = state.counts.cpu().numpy()
        window = [[j] * len(cands) for j in range(J)]
    else:
        p = state.pipe
        off = p.inp.off_host.astype(np.int64)
        keys = p.inp.keys.cpu().numpy()
        rows = np.stack([np.bincount(keys[off[j]:off[j + 1]], minlength=K) for j in range(J)])
        if case["chunk"]:
            rows = np.concatenate([p.prev_counts.cpu().numpy()[None], rows])
        window = np.asarray(p.plan_window).reshape(-1, len(cands)).tolist()
    memo = {}
    load = []
    for row in window:
        for w, c in zip(row, cands):
            key = (w, c.W, c.a, c.b, c.variant, c.place_seed)
            if key not in memo:
                memo[key] = _loads(rows[w], c, R)
            load.append(memo[key])
    load = np.stack(load)
    names = list(_plan_outputs(SimpleNamespace(order=0, order_count=0, n_order=0, num_admitted=0, cold=0, clamped=0,
                                               member_off=0, members=0, load=0, key_index=0, route=0)))
    out = dict.fromkeys(names)
    out["load"] = load
    return out
