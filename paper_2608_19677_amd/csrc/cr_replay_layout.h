// Segment lengths and workspace layout of the replay (cr_replay.hip). Plain arithmetic shared by
// the host, the kernels and a host-only check of the layout.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "../../include/cr.h"

#ifdef __HIPCC__
#define CR_HD __host__ __device__ __forceinline__
#else
#define CR_HD inline
#endif

namespace cr {
namespace {

struct WArg {
    uint16_t W[CR_MAX_CANDS];
    uint8_t grp[CR_MAX_CANDS];  // lists per wavefront: G > 1 for k_replay_grp<G>, else 1
    uint32_t seg_min;  // shortest segment for this call's record count
    uint32_t seg_per;  // records per segment and cache slot, at least
};

// Segments the whole replay is cut into, a few rounds of wavefronts over the chip: a
// wavefront's LRU chain is serial, so several per SIMD hide its latency, and beyond that
// longer segments only save the backward rebuild of the initial state.
constexpr uint64_t kSegTarget = 16384;

// Shortest segments. A call with enough records to fill the chip (kSegFull) cuts nothing
// shorter than kSegFloor records or kSegPerSlot W, so that the rebuild of the initial state
// stays a small part. Smaller calls leave most of the chip idle, and their time is the chain
// of one segment, so they are cut down to kSegShort records or kSegPerSlotShort W, between
// the two in proportion, which keeps about 4,096 wavefronts. One list of 48 slots over 64
// streams: 1e6 requests 61 -> 49 us with segments of 256 instead of 1,024; 4e6 requests 86 us
// with 1,024 and 98 us with 488.
constexpr uint64_t kSegFull = 4u << 20;
constexpr uint32_t kSegFloor = 1024;
constexpr uint32_t kSegCeil = 65536;
constexpr uint32_t kSegShort = 256;
constexpr uint32_t kSegPerSlot = 16;
constexpr uint32_t kSegPerSlotShort = 4;

// The call's shortest segment and its records per cache slot.
inline void seg_rule(uint64_t n, uint32_t P, WArg* wa)
{
    const uint64_t recs = n * P;
    const uint64_t share = (recs + kSegTarget - 1) / kSegTarget;
    const uint32_t floor_ = recs >= kSegFull ? kSegFloor : (uint32_t)(recs * kSegFloor / kSegFull);
    wa->seg_min = share > kSegCeil ? kSegCeil : (uint32_t)share;
    wa->seg_min = wa->seg_min > floor_ ? wa->seg_min : floor_;
    wa->seg_min = wa->seg_min > kSegShort ? wa->seg_min : kSegShort;
    wa->seg_per = recs >= kSegFull ? kSegPerSlot : (uint32_t)(recs * kSegPerSlot / kSegFull);
    wa->seg_per = wa->seg_per > kSegPerSlotShort ? wa->seg_per : kSegPerSlotShort;
}

// Records per segment: at least the call's shortest, seg_per W (the rebuild scans back to W
// distinct keys) and the share that keeps the number of segments near kSegTarget. A candidate
// whose wavefronts hold G lists (k_replay_grp) takes segments G times shorter, so that it
// still has as many wavefronts.
CR_HD uint32_t seg_len(uint32_t W, const WArg& wa, uint32_t G)
{
    uint32_t s = wa.seg_per * W;
    s = s > wa.seg_min ? s : wa.seg_min;
    s = s > kSegCeil ? kSegCeil : s;
    if (G > 1u) s = s / G < kSegFloor ? kSegFloor : s / G;
    return s;
}

// Lists per wavefront of a W-slot list in k_replay_grp (lane groups of 64 / G lanes), or 1
// for the one-wavefront-per-list kernels. Only calls with one interval: the grouped kernel
// keeps one set of statistics per segment. Two lists per wavefront (W <= 32) measured
// slower than one on the 1e8-request sweep (10.2 against 7.2 ms for its W = 26 plans).
constexpr uint32_t kMaxGroup = 8;

CR_HD uint32_t grp_of(uint32_t W, uint32_t J)
{
    if (J != 1u || W > 16u) return 1u;
    return W <= 8u ? kMaxGroup : 4u;
}

struct PartGeom {
    uint64_t tile;
    uint64_t ntiles;
};

inline PartGeom part_geom(uint64_t n, uint32_t P)
{
    const uint64_t target = 16384u / P > 0 ? 16384u / P : 1u;
    uint64_t tile = (n + target - 1) / target;
    tile = (tile + 1023) & ~1023ull;  // whole sub-tiles of the scatter
    if (tile < 1024) tile = 1024;
    return PartGeom{tile, n ? (n + tile - 1) / tile : 0};
}

// Most work items of a call, whatever the slot budgets, the routing and the grouping: a stream
// of cnt records has max(1, ceil(cnt / S)), so a candidate has at most R + n / S, and no
// segment is shorter than one of W = 1, alone or in groups of kMaxGroup (the shorter of the two:
// kSegShort alone against kSegFloor in small calls, kSegCeil against kSegCeil / kMaxGroup in the
// largest).
inline uint64_t max_items(uint64_t n, uint32_t P, uint32_t R)
{
    WArg wa;
    seg_rule(n, P, &wa);
    const uint32_t a = seg_len(1u, wa, 1u), g = seg_len(1u, wa, kMaxGroup);
    return (uint64_t)P * (R + n / (a < g ? a : g));
}

struct ReplayWs {
    uint64_t* rec;
    uint32_t* tcnt;
    uint32_t* dtot;
    uint32_t* grp_off;
    uint32_t* item_off;
    uint32_t* gwave_off;  // [P + 1] first k_replay_grp wavefront of each candidate
    uint8_t* aborted;  // [max_items] byte per work item: its rebuild ran out of budget
    size_t bytes;
};

inline ReplayWs replay_layout(void* base, uint64_t n, uint32_t P, uint32_t R)
{
    const PartGeom g = part_geom(n, P);
    auto up = [](uint64_t x) { return (x + 255) & ~255ull; };
    uint8_t* b = reinterpret_cast<uint8_t*>(base);
    uint64_t o = 0;
    ReplayWs w{};
    w.rec = reinterpret_cast<uint64_t*>(b + o);
    o = up(o + (uint64_t)P * n * 8u);
    w.tcnt = reinterpret_cast<uint32_t*>(b + o);
    o = up(o + (uint64_t)P * R * g.ntiles * 4u);
    w.dtot = reinterpret_cast<uint32_t*>(b + o);
    o = up(o + (uint64_t)P * R * 4u);
    w.grp_off = reinterpret_cast<uint32_t*>(b + o);
    o = up(o + (uint64_t)P * (R + 1u) * 4u);
    w.item_off = reinterpret_cast<uint32_t*>(b + o);
    o = up(o + ((uint64_t)P * R + 1u) * 4u);
    w.gwave_off = reinterpret_cast<uint32_t*>(b + o);
    o = up(o + ((uint64_t)P + 1u) * 4u);
    w.aborted = b + o;
    o = up(o + max_items(n, P, R));
    w.bytes = (size_t)o + 256u;
    return w;
}

}  // namespace
}  // namespace cr
