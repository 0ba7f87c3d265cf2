// Shadow replay of P candidate routings against per-destination LRU prefix caches
// (Section 3.2: admitted and cold prefixes share one cache per destination; Section 3.1
// equal-slot model: W whole-prefix slots per destination).
//
// Pipeline (all on the caller's stream, workspace from the caller):
//   k_part_hist / k_scan_dest / k_seg_items / k_part_scatter64 / k_part_scatter_wide
//        stable partition of every candidate's requests by destination, preserving
//        arrival order; each record packs (key, suffix, interval) into 8 bytes;
//        k_seg_items also splits every (candidate, destination) stream into segments of
//        S records;
//   k_replay
//        one wavefront per segment. The LRU state before a segment is exactly the most
//        recent W distinct keys seen at that destination (carried state appended), so a
//        wavefront rebuilds it by scanning backwards, then replays its segment. This
//        turns R*P sequential streams into thousands of independent wavefronts with
//        results identical to one sequential pass;
//   k_replay_grp<G>
//        lists of at most 16 slots in calls with one interval: G = 4 or 8 segments per
//        wavefront, one per lane group (below).
// Below 64 slots the LRU is a move-to-front list across the lanes of one register: lane i
// holds the i-th most recent key. A lookup is one compare and a ballot; the first set bit p is
// the hit depth, and the update shifts lanes 0..p (all lanes on a miss) up by one and writes
// the key into lane 0, a single select between a lane and its left neighbour under a scalar
// mask. From 64 slots it is a hash table in LDS that takes 64 records per step (below).
#include "cr_common.h"
#include "cr_replay_layout.h"

#include <mutex>

namespace cr {
namespace {

constexpr int kReplayThreads = 256;

// The candidates one k_replay launch serves and the first wavefront of each: wavefront v takes
// work item v - wv0[i] of candidate cand[i] for wv0[i] <= v < wv0[i + 1]. Each
// candidate gets as many wavefronts as it can have work items (one per stream plus one per
// full segment), so a launch runs no wavefront for another list size's candidates. n = 0
// when the launch serves every candidate of the call: wavefront v then takes work item v.
struct CandMap {
    uint32_t n;
    uint16_t cand[CR_MAX_CANDS];
    uint32_t wv0[CR_MAX_CANDS + 1];
};

// Segment i of a stream of cnt records cut into nseg = ceil(cnt / S) segments (at least one):
// records [seg_start(i), seg_start(i + 1)). The stream's ceil(cnt / 64) batches of 64 records
// are dealt evenly, so segments differ by at most one batch and only the last one ends in a
// partial batch (the replay takes a full batch in one unrolled pass, a partial one record by
// record); the wavefronts of a launch thus run for about as long as each other (with
// segments of exactly S, a stream's last one was its remainder, and those short wavefronts
// left the chip part empty near each launch's end). One 32-bit division per bound.
__host__ __device__ __forceinline__ uint32_t seg_start(uint32_t i, uint32_t nseg, uint32_t cnt)
{
    const uint32_t nb = (cnt + 63u) / 64u, L = nb / nseg, r = nb - L * nseg;
    const uint32_t b = i * L + (i < r ? i : r);
    return b < nb ? 64u * b : cnt;
}

// Classes of k_replay: the largest W and the slots of the hash table. Class 0 replays by the
// list in a register; the hash form, in the others, needs W >= 64. Table sizes by measurement, 4e7 requests x 8 candidates over 1,024
// streams: W = 86 2.67 / 2.69 / 2.83 ms with 384 / 512 / 640 slots, W = 156 3.12 / 2.95 / 2.78
// with 512 / 640 / 768, W = 283 3.21 / 3.10 / 3.49 with 768 / 1,024 / 1,280, W = 512 3.93 /
// 3.60 / 3.51 / 3.96 with 1,024 / 1,280 / 1,536 / 2,048: a small table is refreshed more often
// and probes further, a large one leaves fewer wavefronts per CU.
constexpr uint32_t kClasses = 5;
constexpr int kMaxW[kClasses] = {63, 96, 192, 384, 512};
constexpr int kSlots[kClasses] = {256, 384, 768, 1024, 1536};

__host__ __device__ __forceinline__ uint32_t rep_class(uint32_t W)
{
    uint32_t cls = 0;
    while (cls + 1u < kClasses && W > (uint32_t)kMaxW[cls]) ++cls;
    return cls;
}

// Per-tile destination counts; with aligned rows (kVec) every thread reads four
// destinations with one 8-byte load.
constexpr uint32_t kHistThreads = 256;

template <bool kVec>
__global__ __launch_bounds__(kHistThreads) void k_part_hist(const uint16_t* __restrict__ dest, uint64_t n, uint32_t R,
                                                            uint64_t tile, uint64_t ntiles, uint32_t* __restrict__ tcnt,
                                                            uint32_t* __restrict__ err)
{
    issue_priority_high();
    extern __shared__ uint32_t h[];
    const uint32_t c = blockIdx.y;
    const uint64_t t = blockIdx.x;
    const uint64_t t0 = t * tile, t1 = t0 + tile < n ? t0 + tile : n;
    for (uint32_t d = threadIdx.x; d < R; d += blockDim.x) h[d] = 0;
    __syncthreads();
    const uint16_t* __restrict__ dc = dest + (uint64_t)c * n;
    bool bad = false;
    auto add = [&](uint32_t d) {
        if (d < R) atomicAdd(&h[d], 1u);
        else bad = true;
    };
    uint64_t a = t0;
    if (kVec) {
        for (; a + 4u * kHistThreads <= t1; a += 4u * kHistThreads) {
            const uint2 q = *reinterpret_cast<const uint2*>(dc + a + 4u * threadIdx.x);
            add(q.x & 0xFFFFu);
            add(q.x >> 16);
            add(q.y & 0xFFFFu);
            add(q.y >> 16);
        }
    }
    for (uint64_t i = a + threadIdx.x; i < t1; i += blockDim.x) add(dc[i]);
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < R; d += blockDim.x) tcnt[((uint64_t)c * R + d) * ntiles + t] = h[d];
    if (bad) atomicOr(err, CR_ERR_DEST_RANGE);
}

// One block per (destination, candidate): exclusive scan of that destination's per-tile
// counts, which are contiguous in tcnt[c][d][tile], in place; the destination's total goes
// to dtot[c][d]. Destination bases within a candidate are added later (k_seg_items).
constexpr uint32_t kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void k_scan_dest(uint32_t* __restrict__ tcnt, uint64_t ntiles, uint32_t R,
                                                            uint32_t* __restrict__ dtot)
{
    issue_priority_high();
    __shared__ uint32_t s_scan[16];
    const uint32_t d = blockIdx.x, c = blockIdx.y;
    uint32_t* __restrict__ t = tcnt + ((uint64_t)c * R + d) * ntiles;
    uint32_t carry = 0;
    for (uint64_t e0 = 0; e0 < ntiles; e0 += 4u * kScanThreads) {
        const uint64_t e = e0 + 4u * threadIdx.x;
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = e + q < ntiles ? t[e + q] : 0u;
            sum += v[q];
        }
        uint32_t tot;
        uint32_t ex = block_exscan_u32(sum, s_scan, &tot) + carry;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (e + q < ntiles) t[e + q] = ex;
            ex += v[q];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) dtot[(uint64_t)c * R + d] = carry;
}

// The scatter of a tile: stable, into packed records, a sub-tile of requests at a time. Every
// request is ranked among the earlier ones of its destination in the sub-tile; the records are
// then staged in LDS in destination order and written out so that consecutive lanes store
// consecutive addresses of one destination's run: whole cache lines instead of a few bytes in
// each of R streams per instruction.
//
// R <= 64: one wavefront per (tile, candidate), sub-tiles of kSub requests, each lane owning a
// run of kRun consecutive requests of the sub-tile. A lane counts its run's destinations in a
// private row of 16-bit counters in LDS, in request order, which ranks every request within its
// run; a prefix sum of the rows across the lanes (packed pairs of counters, one wave scan per
// pair of destinations) gives each lane's offset per destination. A request's rank within the
// sub-tile is then its lane's offset plus its rank within the run: no cross-lane matching of
// destinations at all. With aligned rows (kVec) a lane reads its run with 16-byte loads.
constexpr uint32_t kSub = 1024;
static_assert(kSub == 1024, "part_geom rounds tiles to 1024 requests");
constexpr uint32_t kRun = kSub / 64;

// Row stride in counters: R in 16-byte pieces, an odd number of them, so that the lanes' pieces
// of one column lie in different banks (at 128 bytes, for R = 64, they all share four).
__host__ __device__ __forceinline__ uint32_t scat64_row(uint32_t R) { return 8u * (((R + 7u) / 8u) | 1u); }

// LDS: the counter rows, and over them, once every request has its slot, the staged records and
// a byte each for their destinations; then two words per destination. 9.7 KB, so that 16
// wavefronts share a CU (21 KB at R = 64 with rows and 4-byte output positions of their own, 7
// wavefronts): the sub-tile's phases are serial and only other wavefronts cover their latency.
// 5e7 requests, 64 destinations: 276 -> 243 us (3.3 TB/s).
constexpr uint32_t kStage64 = kSub * 9u;
static_assert(kStage64 >= 64u * 72u * 2u, "the rows lie under the staged records");
constexpr size_t kScatter64Lds = kStage64 + 64u * 8u;

template <bool kVec>
__global__ __launch_bounds__(64) void k_part_scatter64(const uint32_t* __restrict__ keys,
                                                       const uint16_t* __restrict__ suffix,
                                                       const uint16_t* __restrict__ dest, uint64_t n,
                                                       const uint64_t* __restrict__ off, uint32_t J, uint32_t P, uint32_t R,
                                                       uint64_t tile, uint64_t ntiles, const uint32_t* __restrict__ tcnt,
                                                       const uint32_t* __restrict__ grp_off,
                                                       uint64_t* __restrict__ rec)
{
    issue_priority_high();
    extern __shared__ uint64_t lds[];
    uint64_t* srec = lds;                                            // [kSub] staged records
    uint8_t* sdst = reinterpret_cast<uint8_t*>(srec + kSub);         // [kSub] their destinations
    uint16_t* rows = reinterpret_cast<uint16_t*>(lds);               // [64][RW] counters per lane (until staging)
    uint32_t* sex = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(lds) + kStage64);  // [64] sub-tile offset
    uint32_t* gbase = sex + 64;                                      // [64] output position minus sub-tile offset
    uint32_t* stot = gbase;  // [64] sub-tile count per destination, before
    const uint32_t RW = scat64_row(R), R8 = (R + 7u) & ~7u;
    // an XCD runs the candidates of one tile together (as below for R > 64): the tile's keys
    // and suffixes come from its L2 for all but one of them (2e7 requests x 4 candidates, 16
    // destinations: 300 -> 231 us)
    const uint32_t bi = blockIdx.x / kXcds, c = bi % P, lane = lane_id();
    const uint64_t t = (uint64_t)(bi / P) * kXcds + blockIdx.x % kXcds;
    if (t >= ntiles) return;
    const uint64_t t0 = t * tile, t1 = t0 + tile < n ? t0 + tile : n;
    // lane d: next output position of destination d
    uint32_t run = lane < R ? grp_off[(uint64_t)c * (R + 1u) + lane] + tcnt[((uint64_t)c * R + lane) * ntiles + t] : 0u;
    const uint16_t* __restrict__ dc = dest + (uint64_t)c * n;
    uint64_t* __restrict__ rc = rec + (uint64_t)c * n;
    uint16_t* row = rows + lane * RW;
    uint32_t jw = find_interval(off, J, t0);  // interval of the sub-tile's first request
    for (uint64_t sb = t0; sb < t1; sb += kSub) {
        const uint64_t se = sb + kSub < t1 ? sb + kSub : t1;
        const uint64_t i0 = sb + (uint64_t)lane * kRun;
        uint32_t kv[kRun], dv[kRun], mv[kRun];
        if (kVec && se - sb == kSub) {
            const uint4* k4 = reinterpret_cast<const uint4*>(keys + i0);
            const uint4* d4 = reinterpret_cast<const uint4*>(dc + i0);
            const uint4* m4 = reinterpret_cast<const uint4*>(suffix + i0);
            uint4 qk[4], qd[2], qm[2];
#pragma unroll
            for (uint32_t v = 0; v < 4; ++v) qk[v] = k4[v];
#pragma unroll
            for (uint32_t v = 0; v < 2; ++v) {
                qd[v] = d4[v];
                qm[v] = m4[v];
            }
#pragma unroll
            for (uint32_t v = 0; v < 4; ++v) {
                kv[4 * v + 0] = qk[v].x;
                kv[4 * v + 1] = qk[v].y;
                kv[4 * v + 2] = qk[v].z;
                kv[4 * v + 3] = qk[v].w;
            }
#pragma unroll
            for (uint32_t v = 0; v < 2; ++v) {
                const uint32_t dw[4] = {qd[v].x, qd[v].y, qd[v].z, qd[v].w};
                const uint32_t mw[4] = {qm[v].x, qm[v].y, qm[v].z, qm[v].w};
#pragma unroll
                for (uint32_t h = 0; h < 4; ++h) {
                    dv[8 * v + 2 * h] = dw[h] & 0xFFFFu;
                    dv[8 * v + 2 * h + 1] = dw[h] >> 16;
                    mv[8 * v + 2 * h] = mw[h] & 0xFFFFu;
                    mv[8 * v + 2 * h + 1] = mw[h] >> 16;
                }
            }
        } else {
#pragma unroll
            for (uint32_t v = 0; v < kRun; ++v) {
                const uint64_t i = i0 + v;
                const bool in = i < se;
                dv[v] = in ? dc[i] : 0xFFFFu;
                kv[v] = in ? keys[i] : 0u;
                mv[v] = in ? suffix[i] : 0u;
            }
        }
        for (uint32_t w = 0; w < R8; w += 8) *reinterpret_cast<uint4*>(row + w) = make_uint4(0u, 0u, 0u, 0u);
        // interval of each request: from the sub-tile's, past the boundaries up to it
        uint32_t jl = jw;
        uint64_t nb = jl + 1 < J ? off[jl + 1] : ~0ull;  // first request of the next interval
        // rank of each request within the run: the run's earlier requests to its destination
#pragma unroll
        for (uint32_t v = 0; v < kRun; ++v) {
            const uint64_t i = i0 + v;
            const bool in = i < se;
            while (in && i >= nb) {
                ++jl;
                nb = jl + 1 < J ? off[jl + 1] : ~0ull;
            }
            mv[v] |= jl << 16;
            const uint32_t d = dv[v];
            if (in && d < R) {
                const uint32_t r = row[d];
                row[d] = (uint16_t)(r + 1u);
                dv[v] = d | (r << 16);
            } else {
                dv[v] = 0xFFFFFFFFu;
            }
        }
        // exclusive prefix of the rows across the lanes; lane 63's inclusive sums are the
        // sub-tile's counts per destination
        for (uint32_t w = 0; w < R8; w += 8) {
            uint4* q = reinterpret_cast<uint4*>(row + w);
            const uint4 own = *q;
            const uint4 inc = make_uint4(wave_incl_scan_u32(own.x), wave_incl_scan_u32(own.y),
                                         wave_incl_scan_u32(own.z), wave_incl_scan_u32(own.w));
            *q = make_uint4(inc.x - own.x, inc.y - own.y, inc.z - own.z, inc.w - own.w);
            if (lane == 63) {
                const uint32_t iw[4] = {inc.x, inc.y, inc.z, inc.w};
#pragma unroll
                for (uint32_t h = 0; h < 4; ++h) {
                    stot[w + 2 * h] = iw[h] & 0xFFFFu;
                    stot[w + 2 * h + 1] = iw[h] >> 16;
                }
            }
        }
        __syncthreads();
        // destination offsets within the sub-tile (lane d)
        const uint32_t tl = lane < R ? stot[lane] : 0u;
        const uint32_t ex = wave_incl_scan_u32(tl) - tl;
        const uint32_t total = rdlane(ex + tl, 63);
        sex[lane] = ex;
        __syncthreads();
        gbase[lane] = run - ex;
#pragma unroll
        for (uint32_t v = 0; v < kRun; ++v)
            if (dv[v] != 0xFFFFFFFFu) {
                const uint32_t d = dv[v] & 0xFFFFu;
                dv[v] = d | ((sex[d] + row[d] + (dv[v] >> 16)) << 16);
            }
        __syncthreads();
#pragma unroll
        for (uint32_t v = 0; v < kRun; ++v)
            if (dv[v] != 0xFFFFFFFFu) {
                const uint32_t slot = dv[v] >> 16;
                srec[slot] = (uint64_t)kv[v] | ((uint64_t)mv[v] << 32);
                sdst[slot] = (uint8_t)dv[v];
            }
        __syncthreads();
        for (uint32_t q = lane; q < total; q += 64) rc[gbase[sdst[q]] + q] = srec[q];
        run += tl;
        while (jw + 1 < J && off[jw + 1] <= se) ++jw;  // interval of the next sub-tile's first request
        __syncthreads();
    }
}

// R > 64, several wavefronts per block: sub-tiles of kWideSub requests (1,024 per wavefront),
// wavefront w taking the sub-tile's requests 1024 w .. 1024 w + 1023 as 16 chunks of 64 in
// order. A chunk ranks each request among its chunk's requests to the same destination by a
// matching in LDS; the chunk's leader adds the chunk's count to the wavefront's counter of
// that destination in LDS and hands the old value to its peers, which ranks the request
// within the wavefront's requests. Per destination, a block scan over the totals gives the
// destination's run in the sub-tile and each wavefront's base in it; the records are staged
// in LDS in destination order and written out run by run (about kWideSub / R consecutive
// records per destination).
// Blocks are dealt to the XCDs round-robin; block b takes candidate (b / 8) mod P of tile
// ((b / 8) / P) * 8 + b mod 8, so that an XCD runs the P candidates of one tile together
// and fetches the tile's keys and suffixes into its L2 once for all of them (with the
// candidates fastest over the whole grid, each XCD held eight tiles' keys at a time, more
// than its L2, and read them about once per candidate).
constexpr uint32_t kWideChunks = 16;  // chunks of 64 per wavefront and sub-tile

__host__ __device__ __forceinline__ uint32_t wide_row(uint32_t R) { return (R + 3u) & ~3u; }  // padded to 4 per thread

// The element at p + off + k, for a uniform p and a constant k.
template <typename T>
__device__ __forceinline__ T at_bytes(const T* p, uint32_t off, uint32_t k)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + off + (size_t)k);
}

// LDS: staged keys, suffixes, (with several intervals) intervals and destinations; then 16-bit
// counters per wavefront and destination, which give way to the runs' bases once the records
// are staged. The matching scratch (per wavefront two areas of 64 peer masks and a tag byte per
// destination, one for even and one for odd chunks) and the scan's lie where the records are
// staged later. The phases of a sub-tile are chains of LDS and memory round trips that only
// other wavefronts can cover, and a destination's run in a sub-tile (4 or 8 records at R = 1,024)
// is what a line of HBM gets at once: with one interval, eight wavefronts stage 8,192 records in
// 80 KB, and two blocks share a CU (4 wavefronts per SIMD). The whole partition of 1e8 requests
// x 64 candidates over 1,024 destinations takes 40.6 ms, 47.4 with four wavefronts (74 KB with
// 8-byte records, 32-bit counters and scratch of its own).
template <bool kOne>
__host__ __device__ constexpr uint32_t wide_waves() { return kOne ? 8u : 4u; }

// Blocks of eight wavefronts from which they are used (for one interval): fewer leave CUs idle that
// blocks of four would take. 2e6 requests, 1,024 destinations 41 us with eight and 46 with four;
// 1e6, 65 destinations 32 and 30.
constexpr uint64_t kWideMinBlocks = 128;
static_assert(wide_waves<true>() == 8, "sub-tiles of 8,192");

template <bool kOne>
__host__ __device__ constexpr uint32_t wide_stage_bytes() { return wide_waves<kOne>() * 1024u * (kOne ? 8u : 10u); }

__host__ __device__ __forceinline__ uint32_t wide_area_bytes(uint32_t R) { return 512u + ((wide_row(R) + 8u) & ~7u); }

// (the matching scratch, at most 2 x 1,544 bytes per wavefront, is smaller than the staged records)
template <bool kOne>
inline size_t scatter_wide_lds_bytes(uint32_t R)
{
    return wide_stage_bytes<kOne>() + (size_t)wide_row(R) * 2u * wide_waves<kOne>();
}

template <bool kOne>
__global__ __launch_bounds__(64 * wide_waves<kOne>(), kOne ? 4 : 3) void k_part_scatter_wide(
    const uint32_t* __restrict__ keys, const uint16_t* __restrict__ suffix, const uint16_t* __restrict__ dest,
    uint64_t n, const uint64_t* __restrict__ off, uint32_t J, uint32_t P, uint32_t R,
    uint64_t tile, uint64_t ntiles, const uint32_t* __restrict__ tcnt, const uint32_t* __restrict__ grp_off,
    uint64_t* __restrict__ rec)
{
    constexpr uint32_t kWideWaves = wide_waves<kOne>(), kWideThreads = 64u * kWideWaves, kWideSub = 1024u * kWideWaves;
    constexpr uint32_t kPer = 1024u / kWideThreads, kPairs = kPer / 2u;  // destinations per thread in the scan
    issue_priority_high();
    extern __shared__ uint64_t lds[];
    const uint32_t R4 = wide_row(R), area = wide_area_bytes(R);
    char* base = reinterpret_cast<char*>(lds);
    uint32_t* skey = reinterpret_cast<uint32_t*>(base);              // [kWideSub] staged keys
    uint16_t* sfx = reinterpret_cast<uint16_t*>(skey + kWideSub);    // [kWideSub] their suffixes
    uint16_t* sdst = sfx + kWideSub;                                 // [kWideSub] their destinations
    uint16_t* sivl = sdst + kWideSub;                                // [kWideSub] their intervals (not kOne)
    uint16_t* cnt = reinterpret_cast<uint16_t*>(base + wide_stage_bytes<kOne>());  // [kWideWaves][R4] counts per wavefront, then its slot bases
    uint32_t* gbase = reinterpret_cast<uint32_t*>(cnt);              // [R4] output position of the destination's run minus its start
    uint32_t* s_scan = reinterpret_cast<uint32_t*>(base);
    const uint32_t bi = blockIdx.x / kXcds;
    const uint32_t c = bi % P, lane = lane_id(), wv = wave_in_block(), tid = threadIdx.x;
    // this wavefront's matching scratch: peer masks by representative lane, and a tag byte per
    // destination naming the representative
    unsigned long long* pm0 = reinterpret_cast<unsigned long long*>(base + wv * 2u * area);
    unsigned long long* pm1 = reinterpret_cast<unsigned long long*>(base + wv * 2u * area + area);
    uint8_t* tag0 = reinterpret_cast<uint8_t*>(pm0 + 64);
    uint8_t* tag1 = reinterpret_cast<uint8_t*>(pm1 + 64);
    const uint64_t t = (uint64_t)(bi / P) * kXcds + blockIdx.x % kXcds;
    if (t >= ntiles) return;
    const uint64_t t0 = t * tile, t1 = t0 + tile < n ? t0 + tile : n;
    // thread tid owns destinations kPer tid .. kPer tid + kPer - 1 in the scans: their next output
    // positions
    const bool owner = kPer * tid < R4;
    uint32_t run[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        const uint32_t d = kPer * tid + q;
        run[q] = d < R ? grp_off[(uint64_t)c * (R + 1u) + d] + tcnt[((uint64_t)c * R + d) * ntiles + t] : 0u;
    }
    const uint16_t* __restrict__ dc = dest + (uint64_t)c * n;
    uint64_t* __restrict__ rc = rec + (uint64_t)c * n;
    uint16_t* wc = cnt + wv * R4;
    uint32_t* wc2 = reinterpret_cast<uint32_t*>(wc);  // counter pairs
    for (uint64_t sb = t0; sb < t1; sb += kWideSub) {
        const uint64_t se = sb + kWideSub < t1 ? sb + kWideSub : t1;
        for (uint32_t q = tid; q < kWideWaves * R4 / 4u; q += kWideThreads)
            reinterpret_cast<uint64_t*>(cnt)[q] = 0ull;
        __syncthreads();
        // this wavefront's requests: ws .. ws + 1023 of the sub-tile
        const uint64_t ws = sb + 1024u * wv;
        const uint32_t len = ws < se ? (uint32_t)(se - ws < 1024u ? se - ws : 1024u) : 0u;
        const uint16_t *dw = dc + ws, *xw = suffix + ws;
        const uint32_t* kw = keys + ws;
        uint32_t jl = !kOne && ws < se ? find_interval(off, J, ws) : 0u;
        uint64_t jend = !kOne && jl + 1 < J ? off[jl + 1] : ~0ull;
        uint32_t dk[kWideChunks], kv[kWideChunks], mv[kWideChunks];
        // (uniform bases and 32-bit offsets, and no lane masks for a full 1,024: with them the
        // loads' addresses spill)
        if (len == 1024u) {
#pragma unroll
            for (uint32_t m = 0; m < kWideChunks; ++m) {
                dk[m] = at_bytes(dw, 2u * lane, 128u * m);
                kv[m] = at_bytes(kw, 4u * lane, 256u * m);
                mv[m] = at_bytes(xw, 2u * lane, 128u * m);
            }
        } else {
#pragma unroll
            for (uint32_t m = 0; m < kWideChunks; ++m) {
                dk[m] = 0xFFFFu, kv[m] = 0u, mv[m] = 0u;
                if (64u * m + lane < len) {
                    dk[m] = at_bytes(dw, 2u * lane, 128u * m);
                    kv[m] = at_bytes(kw, 4u * lane, 256u * m);
                    mv[m] = at_bytes(xw, 2u * lane, 128u * m);
                }
            }
        }
        // Chunks in pairs, each with its own matching area, so that the LDS round trips of
        // the two chunks overlap. Lanes with the same destination: every lane writes its id
        // into the destination's tag byte and reads it back, so the lanes of one destination
        // read one common representative (whichever write landed last); each lane then sets
        // its bit in the representative's peer mask and reads the mask. LDS operations of a
        // wavefront complete in order, so no barrier is needed, and the counter updates of
        // chunk m precede those of chunk m + 1; the fences keep the compiler from answering a
        // lane's read with the value the lane itself stored.
#pragma unroll
        for (uint32_t m = 0; m < kWideChunks; m += 2) {
            uint32_t dd[2], jj[2];
            bool vv[2];
#pragma unroll
            for (uint32_t h = 0; h < 2; ++h) {
                const uint64_t base = ws + 64u * (m + h);
                dd[h] = dk[m + h];
                vv[h] = dd[h] < R;  // (0xFFFF past the end)
                uint32_t j = jl;
                if (!kOne && base < se && base + 63 >= jend) {  // an interval boundary falls inside these 64
                    while (j + 1 < J && off[j + 1] <= base + lane) ++j;
                    jl = rdlane(j, 63);
                    jend = jl + 1 < J ? off[jl + 1] : ~0ull;
                }
                jj[h] = j;
            }
            pm0[lane] = 0ull;
            pm1[lane] = 0ull;
            // (a lane without a destination takes the tag byte past the last one and counts nothing)
            const uint32_t b0 = vv[0] ? dd[0] : R4, b1 = vv[1] ? dd[1] : R4;
            tag0[b0] = (uint8_t)lane;
            tag1[b1] = (uint8_t)lane;
            wave_lds_fence();
            const uint32_t rep0 = tag0[b0], rep1 = tag1[b1];
            atomicOr(&pm0[rep0], 1ull << lane);
            atomicOr(&pm1[rep1], 1ull << lane);
            wave_lds_fence();
            const uint64_t peers0 = pm0[rep0], peers1 = pm1[rep1];
            const uint32_t rk0 = mbcnt64(peers0), rk1 = mbcnt64(peers1);
            const uint32_t ld0 = (uint32_t)__builtin_ctzll(peers0), ld1 = (uint32_t)__builtin_ctzll(peers1);
            uint32_t old0 = 0, old1 = 0;
            const uint32_t h0 = (b0 & 1u) * 16u, h1 = (b1 & 1u) * 16u;
            if (vv[0] && rk0 == 0) old0 = (atomicAdd(&wc2[b0 >> 1], (uint32_t)__popcll(peers0) << h0) >> h0) & 0xFFFFu;
            if (vv[1] && rk1 == 0) old1 = (atomicAdd(&wc2[b1 >> 1], (uint32_t)__popcll(peers1) << h1) >> h1) & 0xFFFFu;
            old0 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(ld0 << 2), (int)old0);
            old1 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(ld1 << 2), (int)old1);
            dk[m] = vv[0] ? (dd[0] << 16) | (old0 + rk0) : 0xFFFFFFFFu;  // destination, rank in the wavefront
            dk[m + 1] = vv[1] ? (dd[1] << 16) | (old1 + rk1) : 0xFFFFFFFFu;
            asm volatile("" : "+v"(dk[m]), "+v"(dk[m + 1]));  // (formed here, not from its parts where it is used)
            if (!kOne) {
                mv[m] |= jj[0] << 16;
                mv[m + 1] |= jj[1] << 16;
            }
            wave_lds_fence();
        }
        __syncthreads();
        // destination runs in the sub-tile: each wavefront's slot base within its destination's
        // run, and the run's output position minus its start
        uint32_t cw[kWideWaves][kPairs];
        uint32_t tq[kPer] = {}, sum = 0;
        if (owner)
#pragma unroll
            for (uint32_t w = 0; w < kWideWaves; ++w)
#pragma unroll
                for (uint32_t h = 0; h < kPairs; ++h) {
                    const uint32_t x = reinterpret_cast<const uint32_t*>(cnt + w * R4 + kPer * tid)[h];
                    cw[w][h] = x;
                    tq[2 * h] += x & 0xFFFFu, tq[2 * h + 1] += x >> 16;
                }
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) sum += tq[q];
        uint32_t total;
        uint32_t acc = block_exscan_u32(sum, s_scan, &total);
        uint32_t gb[kPer];
        if (owner) {
#pragma unroll
            for (uint32_t h = 0; h < kPairs; ++h) {
                uint32_t b0 = acc, b1 = acc + tq[2 * h];  // bases are below kWideSub
                gb[2 * h] = run[2 * h] - b0, gb[2 * h + 1] = run[2 * h + 1] - b1;
                run[2 * h] += tq[2 * h], run[2 * h + 1] += tq[2 * h + 1];
                acc = b1 + tq[2 * h + 1];
#pragma unroll
                for (uint32_t w = 0; w < kWideWaves; ++w) {
                    const uint32_t x = cw[w][h];
                    reinterpret_cast<uint32_t*>(cnt + w * R4 + kPer * tid)[h] = b0 | (b1 << 16);
                    b0 += x & 0xFFFFu, b1 += x >> 16;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t m = 0; m < kWideChunks; ++m) {
            if (dk[m] != 0xFFFFFFFFu) {
                const uint32_t d = dk[m] >> 16, lr = dk[m] & 0xFFFFu;
                const uint32_t slot = wc[d] + lr;
                skey[slot] = kv[m];
                sfx[slot] = (uint16_t)mv[m];
                sdst[slot] = (uint16_t)d;
                if (!kOne) sivl[slot] = (uint16_t)(mv[m] >> 16);
            }
        }
        __syncthreads();
        if (owner)
#pragma unroll
            for (uint32_t q = 0; q < kPer; ++q) gbase[kPer * tid + q] = gb[q];
        __syncthreads();
        for (uint32_t q = tid; q < total; q += kWideThreads) {
            const uint32_t hi = kOne ? (uint32_t)sfx[q] : (uint32_t)sfx[q] | ((uint32_t)sivl[q] << 16);
            rc[gbase[sdst[q]] + q] = (uint64_t)skey[q] | ((uint64_t)hi << 32);
        }
        __syncthreads();
    }
}

// Destination bases and work items, from the destination totals dtot[c][d]:
//   grp_off[c][d] = records of candidate c routed to destinations < d (grp_off[c][R] = all),
//   item_off[e]   = first work item of stream e = c * R + d, one item per segment of S
//                   records (at least one per stream).
// Pass one scans over all (c, d) in one block; pass two rebases grp_off per candidate.
__global__ __launch_bounds__(1024) void k_seg_items(const uint32_t* __restrict__ dtot, uint32_t P, uint32_t R,
                                                    WArg wa, uint32_t* __restrict__ grp_off,
                                                    uint32_t* __restrict__ item_off, uint32_t* __restrict__ gwave_off)
{
    issue_priority_high();
    __shared__ uint32_t s_scan[16];
    __shared__ uint32_t s_cstart[CR_MAX_CANDS + 1];
    const uint32_t total = P * R;
    uint32_t carry = 0, icarry = 0;
    for (uint32_t e0 = 0; e0 < total; e0 += blockDim.x) {
        const uint32_t e = e0 + threadIdx.x;
        uint32_t cnt = 0, nseg = 0;
        if (e < total) {
            cnt = dtot[e];
            const uint32_t S = seg_len(wa.W[e / R], wa, wa.grp[e / R]);
            nseg = cnt ? (cnt + S - 1) / S : 1u;
        }
        uint32_t tot, itot;
        const uint32_t ex = block_exscan_u32(cnt, s_scan, &tot);
        const uint32_t iex = block_exscan_u32(nseg, s_scan, &itot);
        if (e < total) {
            const uint32_t c = e / R, d = e % R;
            grp_off[(uint64_t)c * (R + 1u) + d] = carry + ex;
            item_off[e] = icarry + iex;
            if (d == 0) s_cstart[c] = carry + ex;
        }
        carry += tot;
        icarry += itot;
    }
    if (threadIdx.x == 0) {
        item_off[total] = icarry;
        s_cstart[P] = carry;
    }
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < total; e += blockDim.x) {
        const uint32_t c = e / R, d = e % R;
        grp_off[(uint64_t)c * (R + 1u) + d] -= s_cstart[c];
    }
    for (uint32_t c = threadIdx.x; c < P; c += blockDim.x)
        grp_off[(uint64_t)c * (R + 1u) + R] = s_cstart[c + 1] - s_cstart[c];
    // gwave_off[c]: first k_replay_grp wavefront of candidate c (G work items per wavefront;
    // none for candidates replayed one list per wavefront)
    __syncthreads();
    const uint32_t c = threadIdx.x;
    const uint32_t G = c < P ? wa.grp[c] : 1u;
    const uint32_t nw = G > 1u ? (item_off[(c + 1u) * R] - item_off[c * R] + G - 1u) / G : 0u;
    uint32_t wtot;
    const uint32_t wex = block_exscan_u32(nw, s_scan, &wtot);  // P <= CR_MAX_CANDS <= blockDim.x
    if (c < P) gwave_off[c] = wex;
    if (c == 0) gwave_off[P] = wtot;
}

// Move-to-front update after a lookup whose hit mask is m: p = first set bit of m
// (0xFFFFFFFF when none); lanes 1..p (every lane on a miss) take their left neighbour's
// key and deeper lanes keep theirs, by one v_cndmask with a wave_shr:1 DPP source under
// VCC = ~1 << p. Lane 0 is left undefined for the caller to overwrite with the key. The
// scalar steps sit in the same block as the select so that no wait states are inserted
// between them; the DPP read of sk comes at least three instructions after sk's last
// VALU write (the compare that produced m, s_ff1 and s_lshl), which covers the two wait
// states such a read needs.
__device__ __forceinline__ uint32_t mtf_core(uint32_t& sk, uint64_t m)
{
    uint32_t p, out;
    asm("s_ff1_i32_b64 %1, %3\n\t"
        "s_lshl_b64 vcc, -2, %1\n\t"
        "v_cndmask_b32_dpp %0, %2, %2, vcc wave_shr:1 row_mask:0xf bank_mask:0xf"
        : "=v"(out), "=&s"(p)
        : "v"(sk), "s"(m)
        : "vcc", "scc");  // s_lshl_b64 sets SCC
    sk = out;
    return p;
}

// Move-to-front access of key kk (lane i = i-th most recent key; lanes outside `wmask`
// are ignored). Returns the hit depth, or 0xFFFFFFFF on a miss. On a miss the shift runs
// over every lane, which drops the least recent key of a full list.
__device__ __forceinline__ uint32_t mtf_step(uint32_t& sk, uint32_t kk, uint64_t wmask)
{
    const uint32_t p = mtf_core(sk, ballot(sk == kk) & wmask);
    sk = wrlane(sk, kk, 0u);
    return p;
}

// 64 records (all valid) through the move-to-front list; returns lane t = hit depth of record
// t. The keys come from the batch's records (rb is uniform) by scalar loads, 8 records per
// load: no vector instruction moves a key into a scalar register, and the other wavefronts of
// the SIMD cover the wait for each load.
__device__ __forceinline__ uint32_t mtf_batch(uint32_t& sk, const uint64_t* __restrict__ rb, uint64_t wmask)
{
    uint32_t depth = 0xFFFFFFFFu;
#pragma unroll
    for (uint32_t g = 0; g < 8; ++g) {
        uint32_t key[8];
#pragma unroll
        for (uint32_t t = 0; t < 8; ++t) key[t] = (uint32_t)rb[8u * g + t];
#pragma unroll
        for (uint32_t t = 0; t < 8; ++t) {
            const uint32_t p = mtf_core(sk, ballot(sk == key[t]) & wmask);
            sk = wrlane(sk, key[t], 0u);
            depth = wrlane(depth, p, 8u * g + t);
        }
    }
    return depth;
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v)
{
    if (ballot((v >> 26) != 0ull) == 0ull) return rdlane(wave_incl_scan_u32((uint32_t)v), 63u);  // the sum fits 32 bits
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += (uint64_t)__shfl_xor((unsigned long long)v, o, 64);
    return v;
}

// Statistics of one stream: per-lane sums for the current interval, flushed (one atomic per
// statistic) when the interval changes and at the end of a range.
struct StreamStats {
    uint64_t* __restrict__ stats;
    uint32_t P, R, J, c, d, lane;
    uint32_t cur = 0xFFFFFFFFu;
    uint32_t n_req = 0, n_hit = 0;  // uniform: a wavefront replays fewer than 2^32 records
    uint64_t a_pre = 0, a_hp = 0;

    __device__ __forceinline__ void flush()
    {
        if (cur >= J) return;
        const uint64_t r2 = wave_sum_u64(a_pre), r3 = wave_sum_u64(a_hp);
        if (lane == 0) {
            unsigned long long* st = (unsigned long long*)(stats + (((uint64_t)cur * P + c) * R + d) * 4u);
            atomicAdd(st + 0, (unsigned long long)n_req);
            if (n_hit) atomicAdd(st + 1, (unsigned long long)n_hit);
            atomicAdd(st + 2, (unsigned long long)r2);
            if (r3) atomicAdd(st + 3, (unsigned long long)r3);
        }
        n_req = n_hit = 0;
        a_pre = a_hp = 0;
    }

    // The records of the lanes of vm: record word, the lanes that hit, the keys' prefix lengths.
    __device__ __forceinline__ void add(uint64_t rv, uint64_t vm, uint64_t hm, uint32_t pl)
    {
        const uint32_t sfx = (uint32_t)(rv >> 32) & 0xFFFFu;
        const uint32_t ivl = (uint32_t)(rv >> 48);
        const bool hl = __builtin_amdgcn_inverse_ballot_w64(hm);
        while (vm) {
            const uint32_t iv = rdlane(ivl, first_lane(vm));
            if (iv != cur) {
                flush();
                cur = iv;
            }
            const uint64_t sel = vm & ballot(ivl == iv);
            n_req += (uint32_t)__popcll(sel);
            n_hit += (uint32_t)__popcll(sel & hm);
            if (__builtin_amdgcn_inverse_ballot_w64(sel)) {
                a_pre += (uint64_t)sfx + (hl ? 0u : pl);
                a_hp += hl ? pl : 0u;
            }
            vm &= ~sel;
        }
    }
};

// One work item per segment (kSeq false), or per run of consecutive segments whose
// rebuild ran out of budget (kSeq true).
//
// A segment rebuilds its initial state by scanning back for W distinct keys; a stream with
// fewer distinct keys than W would make every segment scan to the stream's start, which is
// quadratic in its length. The scan therefore stops after kRebuildBudget segment lengths:
// a segment that has neither found W keys nor reached the start writes nothing and marks
// itself in `aborted`. In the kSeq launch that follows, the wavefront of the first segment
// of each run of marked segments starts at the run's predecessor (which is never marked:
// the first segment of a stream has nothing to rebuild), rebuilds the predecessor's state
// as that segment did, replays it without counting, and then replays the run in order,
// counting it and writing the final state if the run ends the stream. Each marked record
// is thus replayed once more, and every record is scanned at most kRebuildBudget + 1 times
// (by segments of S < kSegFloor records, kRebuildBudget kSegFloor / S + 1 times), whatever the keys. The kSeq launch rebuilds without a budget: a run's predecessor is an
// unmarked segment, whose rebuild ended within its budget. A scan that meets known keys only
// takes 256 records a step, about a tenth of the time their replay takes, and a marked run is
// one serial chain, so the budget is wide: 2,000 keys over 30 streams of 133,000 requests took
// 1.40, 0.69 and 0.30 ms at W = 512 with budgets of 8, 32 and 64 segment lengths (1.74, 1.58
// and 1.31 ms at W = 100); streams that fill their caches never come near it.
constexpr uint32_t kRebuildBudget = 64;

// Records the backward rebuild of a segment of length S may scan (of segments cut shorter
// than kSegFloor, as many as of those).
__device__ __forceinline__ uint32_t rebuild_budget(uint32_t S) { return kRebuildBudget * (S > kSegFloor ? S : kSegFloor); }

// Budget of k_replay_grp's forward rebuild, in its own (G times shorter) segment lengths.
// Its rebuild windows run in lockstep with the other lists of the wavefront, so a deep one
// holds up G - 1 others: with eight, the 1e8-request sweep's W = 8 and 14 plans took 15.6 ms
// against 12.7 ms with two (kSeq pass included).
constexpr uint32_t kGrpRebuildBudget = 2;

// Marks: one byte per work item, which the item's wavefront of the first pass writes (1: its
// rebuild ran out of budget, and the kSeq pass replays it).
__device__ __forceinline__ bool item_marked(const uint8_t* __restrict__ aborted, uint64_t it) { return aborted[it] != 0u; }

// ---------------------------------------------------------------------------------------
// Lists of 64 slots and more: 64 records per step instead of one. A wavefront keeps the
// segment's cache as a hash table in LDS, {key, position of its last access}, where newer
// accesses have smaller positions, and a bitmap over the positions that marks the last access
// of every cached key. The cache is the table's entries at positions up to T, T being the
// position of the W-th most recent key; a key's depth in the list is the number of bits below
// its position. A step takes 64 records, one per lane:
//   - every lane finds its key in the table or claims a slot for it;
//   - with W >= 64, a key seen earlier in the step is always a hit (at most 62 other keys lie
//     between). A key seen here first is a hit iff it was cached and was not pushed out earlier
//     in the step: at depth d it is still there after c other keys iff d + c < W, where only
//     the keys that were behind it (deeper or not cached) count, each once. Only lanes with
//     d + 63 >= W can fail that; those that the counts of all such keys before them do not
//     decide are counted exactly, one ballot each;
//   - the step's last access of every key becomes its position, the old position's bit is
//     cleared, and T moves to the W-th bit.
// The cost of a step hardly depends on W, where a list in registers paid a compare and a move
// per 64 slots for every record. Measured (the cr_replay_lru call, 4e7 Zipf 0.9 requests of 1e6
// keys x 8 candidates over 1,024 streams, four in five routed by key; list in registers before):
// W = 64 3.26 -> 2.31 ms, 86 5.58 -> 2.43, 156 6.89 -> 2.52, 283 9.98 -> 2.92, 512 16.7 -> 4.22.
// Bound by instruction issue where many wavefronts fit a SIMD and by the latency of the
// dependent LDS round trips where the tables leave few: counters of 8e8 records give, at W = 86,
// 156, 283 and 512, 5.6, 4.1, 3.2 and 2.1 wavefronts per SIMD, VALU busy 0.59, 0.56, 0.49 and 0.37 of
// the time and wavefronts waiting 0.39 to 0.52 of theirs; the list of W < 64 keeps the VALU busy 0.80.
// Entries past T stay in the table (their keys may come back to the same slot); when the
// table or the 64 bitmap words run full, the live entries are re-inserted into an empty table
// at positions that leave the words before them free (refresh).
template <int NS, int kMaxW>
struct HashLds {
    uint4 tab[NS / 2];            // buckets of two {key, position}
    unsigned long long bm[64];    // word b: positions 64 b .. 64 b + 63
    uint32_t list[kMaxW];         // keys or entries by depth, for refresh and rebuild
};

constexpr uint32_t kNoPos = 4096u;     // position of an entry that is not cached
constexpr uint32_t kMarkPos = 8192u;   // above it: marks of the lanes of one step

__device__ __forceinline__ uint32_t bperm(uint32_t src_lane, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src_lane << 2), (int)v);
}

__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

__device__ __forceinline__ void clear_bit(uint64_t& m, uint32_t t) { asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(t)); }

// One wavefront's cache. Masks of lanes and all members but w, pex and inc are uniform.
template <int NS, int kMaxW>
struct HashCache {
    static_assert(NS % 128 == 0 && kMaxW + 128 <= NS * 7 / 8, "whole LDS rounds; room for two steps of claims past a full cache");
    HashLds<NS, kMaxW>& lds;
    uint32_t W, lane;
    uint32_t used = 0;        // claimed slots
    uint32_t live = 0;        // cached keys
    int32_t beta = 63;        // bitmap word of the next step (below every word in use)
    uint32_t T = kNoPos - 1;  // entries at positions past T are not cached
    uint64_t w = 0;           // lane b: bitmap word b
    uint32_t pex = 0;         // lane b: live positions in the words before b
    uint32_t inc = 0;         // lane b: the same with word b

    __device__ __forceinline__ HashCache(HashLds<NS, kMaxW>& l, uint32_t W_, uint32_t lane_) : lds(l), W(W_), lane(lane_) {}

    // The 32-bit word at byte address a of the table (an entry's key; its position is at a + 4).
    __device__ __forceinline__ uint32_t* at(uint32_t a)
    {
        return reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(lds.tab) + a);
    }

    __device__ __forceinline__ void clear()
    {
#pragma unroll 4
        for (uint32_t i = 0; i < NS / 2u; i += 64u) lds.tab[i + lane] = make_uint4(CR_EMPTY_SLOT, kNoPos, CR_EMPTY_SLOT, kNoPos);
        used = 0;
        wave_lds_fence();
    }

    // Byte address of the entry of every lane's key (lanes of am), claimed if the table does
    // not hold it; `pos` = the entry's position (kNoPos when claimed here). Entries are
    // claimed in probe order, so a lookup ends at the key or at a bucket with its second slot
    // empty. The lanes of one key take the same path, so a key never gets two entries; the
    // table always has an empty slot, so every probe ends.
    __device__ __forceinline__ uint32_t find(uint32_t key, uint64_t am, uint32_t& pos)
    {
        uint32_t a = __umulhi(key * 0x9E3779B1u, NS / 2u) * 16u;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        uint64_t todo = am;
        while (todo) {  // a lane's v and a stay as they are once it is done
            if (lane_in(todo)) v = *reinterpret_cast<const uint4*>(at(a));
            todo = ballot(v.x != key) & ballot(v.z != key) & ballot(v.z != CR_EMPTY_SLOT) & am;
            const uint32_t next = a + 16u;
            a = lane_in(todo) ? (next < NS * 8u ? next : 0u) : a;
        }
        const bool h0 = v.x == key, h1 = v.z == key;
        pos = h0 ? v.y : (h1 ? v.w : kNoPos);
        a += h0 || (!h1 && v.x == CR_EMPTY_SLOT) ? 0u : 8u;
        todo = am & ~(ballot(h0) | ballot(h1));
        uint32_t claimed = 0, prev = 0;
        while (todo) {
            if (lane_in(todo)) prev = atomicCAS(at(a), CR_EMPTY_SLOT, key);
            const uint64_t won = ballot(prev == CR_EMPTY_SLOT) & todo;
            claimed += (uint32_t)__popcll(won);
            todo = todo & ~won & ballot(prev != key);  // another key took it: the next slot
            const uint32_t next = a + 8u;
            a = lane_in(todo) ? (next < NS * 8u ? next : 0u) : a;
        }
        used += claimed;
        wave_lds_fence();
        return a;
    }

    // Depth in the list of a cached key at position `p`.
    __device__ __forceinline__ uint32_t depth_of(uint32_t p) const
    {
        const uint32_t wd = (p >> 6) & 63u;
        const uint32_t lo = bperm(wd, (uint32_t)w), hi = bperm(wd, (uint32_t)(w >> 32));
        return bperm(wd, pex) + (uint32_t)__popcll((((uint64_t)hi << 32) | lo) & ~(~0ull << (p & 63u)));
    }

    // Visits every cached key as f(key, depth).
    template <typename F>
    __device__ __forceinline__ void each_live(F f)
    {
        for (uint32_t i = 0; i < (uint32_t)NS; i += 64u) {
            const uint2 e = *reinterpret_cast<const uint2*>(at(8u * (i + lane)));
            const uint32_t d = depth_of(e.y);
            if (e.y <= T) f(e.x, d);
        }
    }

    // The cache made of the n entries whose byte addresses lds.list holds, list[i] at depth i.
    __device__ __forceinline__ void place(uint32_t n)
    {
        const uint32_t w0 = 64u - ((n + 63u) >> 6);  // first bitmap word in use
        for (uint32_t i = lane; i < n; i += 64u) at(lds.list[i])[1] = 64u * w0 + i;
        live = n;
        T = kNoPos - 1u;
        beta = (int32_t)w0 - 1;
        const uint32_t b = lane >= w0 ? 64u * (lane - w0) : n;  // positions before this lane's word
        const uint32_t c = n - b < 64u ? n - b : 64u;
        w = lane < w0 || c == 0u ? 0ull : (c == 64u ? ~0ull : (1ull << c) - 1ull);
        pex = lane >= w0 ? b : 0u;
        inc = lane >= w0 ? b + c : 0u;
        lds.bm[lane] = w;
        wave_lds_fence();
    }

    __device__ __forceinline__ void refresh()
    {
        each_live([&](uint32_t key, uint32_t d) { lds.list[d] = key; });
        wave_lds_fence();
        clear();
        for (uint32_t i0 = 0; i0 < live; i0 += 64u) {
            const uint32_t i = i0 + lane;
            const bool in = i < live;
            uint32_t pos;
            const uint32_t a = find(in ? lds.list[i] : 0u, ballot(in), pos);
            if (in) lds.list[i] = a;
            wave_lds_fence();
        }
        place(live);
    }

    // One step: 64 records in lane order, key kk on the lanes of am. Returns the lanes that hit.
    __device__ __forceinline__ uint64_t step(uint32_t kk, uint64_t am)
    {
        if (beta < 0 || used + 64u > (uint32_t)NS * 7u / 8u) refresh();
        uint32_t old;
        uint32_t* __restrict__ e = at(find(kk, am, old)) + 1;
        const bool act = lane_in(am);
        // the step's first and last record of every key
        const uint32_t c0 = kMarkPos + 63u - lane, c1 = 64u * (uint32_t)beta + 63u - lane;
        if (act) atomicMax(e, c0);
        wave_lds_fence();
        const uint64_t fm = ballot(*e == c0) & am;
        wave_lds_fence();
        uint64_t lm = fm;
        if (fm == am) {  // no key twice
            if (act) *e = c1;
        } else {
            if (act) atomicMin(e, c1);
            wave_lds_fence();
            lm = ballot(*e == c1) & am;
        }
        wave_lds_fence();
        // hits; the lanes that may have been pushed out in this step are counted
        const uint64_t pm = ballot(old <= T) & am;  // cached before the step
        uint64_t hits = am & ~(fm & ~pm);
        const uint32_t nw = (uint32_t)__popcll(ballot(inc + 63u <= W));  // words wholly at depths below W - 63
        const uint64_t near = fm & ballot(old >= 64u * nw) & pm;
        if (near) {
            const uint64_t absent = fm & ~pm;
            const uint32_t d = depth_of(old);
            const uint64_t out = ballot(d + mbcnt64(absent) >= W) & near;
            uint64_t open = ballot(d + mbcnt64(absent | near) >= W) & near & ~out;
            hits &= ~out;
            const uint32_t key = lane_in(pm) ? old : kNoPos;  // absent keys are behind every cached one
            while (open) {
                const uint32_t t = first_lane(open);
                const uint64_t ahead = ballot(key > rdlane(old, t)) & fm & ~(~0ull << t);
                if (rdlane(d, t) + (uint32_t)__popcll(ahead) >= W) clear_bit(hits, t);
                clear_bit(open, t);
            }
        }
        // positions: the old ones out, the step's own in
        if (lane_in(lm & pm)) atomicXor(reinterpret_cast<uint32_t*>(lds.bm) + (old >> 5), 1u << (old & 31u));
        wave_lds_fence();
        w = lds.bm[lane];
        const uint64_t own = __builtin_bitreverse64(lm);
        w = (uint64_t)wrlane((uint32_t)w, (uint32_t)own, (uint32_t)beta) |
            ((uint64_t)wrlane((uint32_t)(w >> 32), (uint32_t)(own >> 32), (uint32_t)beta) << 32);
        const uint32_t c = (uint32_t)__popcll(w);
        inc = wave_incl_scan_u32(c);
        pex = inc - c;
        live = rdlane(inc, 63);
        --beta;
        if (live > W) {  // push out what is past the W-th
            const uint32_t wl = (uint32_t)__popcll(ballot(inc < W));  // word of the W-th
            const uint64_t ww = rdlane64(w, wl);
            const uint32_t b = first_lane(ww & ballot(mbcnt64(ww) + rdlane(pex, wl) == W - 1u));
            T = 64u * wl + b;
            const uint64_t keep = ~(~0ull << b << 1);
            w = lane > wl ? 0ull : (lane == wl ? w & keep : w);
            inc = inc < W ? inc : W;
            live = W;
        }
        lds.bm[lane] = w;
        wave_lds_fence();
        return hits;
    }

    // Rebuild: the next older records (the lanes' order is the stream's). The entries of keys
    // not met yet are appended to lds.list, newest first; q counts them (those past W, which
    // only the last rebuild step can meet, stay in the table as not cached).
    __device__ __forceinline__ uint32_t rebuild_step(uint32_t kk, uint64_t am, uint32_t q)
    {
        uint32_t pos;
        const uint32_t a = find(kk, am, pos);
        uint32_t* __restrict__ e = at(a) + 1;
        const uint64_t fresh = ballot(pos == kNoPos) & am;
        if (lane_in(fresh)) atomicMax(e, kMarkPos + lane);
        wave_lds_fence();
        const uint64_t rep = ballot(*e == kMarkPos + lane) & fresh;  // its newest record here
        wave_lds_fence();
        const uint32_t total = (uint32_t)__popcll(rep);
        const uint32_t i = q + total - 1u - mbcnt64(rep);
        if (lane_in(rep)) {
            *e = i < W ? 0u : kNoPos;
            if (i < W) lds.list[i] = a;
        }
        wave_lds_fence();
        return q + total;
    }

    // Whether every key of k[0..3] (lanes of am[0..3]) is in the table: four lookups in flight.
    __device__ __forceinline__ bool all_known(const uint32_t (&k)[4], const uint64_t (&am)[4])
    {
        uint32_t a[4];
        uint4 v[4];
        uint64_t todo[4], any = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = __umulhi(k[u] * 0x9E3779B1u, NS / 2u) * 16u;
            v[u] = *reinterpret_cast<const uint4*>(at(a[u]));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            todo[u] = ballot(v[u].x != k[u]) & ballot(v[u].z != k[u]) & am[u];
            any |= todo[u];
        }
        while (any) {  // the next bucket, unless this one ends the probe
            any = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (todo[u] & ballot(v[u].z == CR_EMPTY_SLOT)) return false;
                const uint32_t next = a[u] + 16u;
                a[u] = lane_in(todo[u]) ? (next < NS * 8u ? next : 0u) : a[u];
                v[u] = *reinterpret_cast<const uint4*>(at(a[u]));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                todo[u] = ballot(v[u].x != k[u]) & ballot(v[u].z != k[u]) & am[u];
                any |= todo[u];
            }
        }
        return true;
    }

    // The entries of the W most recent distinct keys of records [0, s0) of the stream rl into
    // lds.list, newest first; q counts the distinct keys met. Records are read backwards 64 at
    // a time, the next (older) batch in flight while one is scanned; after a batch that brought
    // no new key, 256 at a time for as long as they bring none. False if `budget` records ran
    // out with fewer than W keys and records left.
    __device__ __forceinline__ bool rebuild(const uint64_t* __restrict__ rl, uint32_t s0, uint32_t K, uint32_t budget,
                                            uint32_t& q)
    {
        uint32_t pos = s0;
        const uint32_t stop = s0 > budget ? s0 - budget : 0u;
        while (q < W && pos > stop) {
            bool none = false;
            uint32_t nb = pos < 64u ? pos : 64u;
            uint32_t next = lane < nb ? (uint32_t)rl[pos - nb + lane] : CR_EMPTY_SLOT;
            while (q < W && pos > stop && !none) {
                const uint32_t kl = next;
                pos -= nb;
                nb = pos < 64u ? pos : 64u;
                next = lane < nb ? (uint32_t)rl[pos - nb + lane] : CR_EMPTY_SLOT;
                const uint32_t was = q;
                q = rebuild_step(kl, ballot(kl < K), q);
                none = q == was;
            }
            bool known = q < W && pos >= 256u && pos > stop;
            uint32_t kn[4];
            if (known)
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) kn[u] = (uint32_t)rl[pos - 256u + 64u * u + lane];
            while (known) {
                uint32_t k[4];
                uint64_t am[4];
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    k[u] = kn[u];
                    am[u] = ballot(k[u] < K);
                }
                const bool more = pos >= 512u;
                if (more)
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u) kn[u] = (uint32_t)rl[pos - 512u + 64u * u + lane];
                if (!all_known(k, am)) break;
                pos -= 256u;
                known = more && pos > stop;
            }
        }
        return q >= W || pos == 0u;
    }

    // The same over a carried state row, newest first and up to its first empty entry.
    __device__ __forceinline__ void rebuild_carried(const uint32_t* __restrict__ li, uint32_t K, uint32_t& q)
    {
        for (uint32_t s = 0; s < W && q < W; s += 64) {
            const uint32_t i = s + 63u - lane;  // lane 63 takes the newest of 64 entries
            const uint32_t kk = i < W ? li[i] : CR_EMPTY_SLOT;
            const uint64_t empty = ballot(kk == CR_EMPTY_SLOT);
            const uint64_t valid = empty ? ~0ull << (63u - (uint32_t)__builtin_clzll(empty)) : ~0ull;
            q = rebuild_step(kk, ballot(kk < K) & valid, q);
            if (empty) break;
        }
    }
};

// One wavefront per segment (or run of marked segments), of candidates with kMinW <= W <= kMaxW.
// With kList the cache is the list in a register and the hash table serves the rebuild alone.
// At most 96 scalar registers, so that eight wavefronts fit on a SIMD.
template <int NS, int kMinW, int kMaxW, bool kList, bool kSeq>
__global__ __launch_bounds__(64) __attribute__((amdgpu_num_sgpr(96))) void k_replay(
    const uint64_t* __restrict__ rec, uint64_t n, const uint32_t* __restrict__ grp_off,
    const uint32_t* __restrict__ item_off, uint32_t P, uint32_t R, uint32_t K, uint32_t J,
    const uint32_t* __restrict__ prefix_len, WArg wa, CandMap cm, uint32_t max_W,
    const uint32_t* __restrict__ lru_in, uint32_t* __restrict__ lru_out, uint64_t* __restrict__ stats,
    uint8_t* __restrict__ aborted, uint32_t* __restrict__ err)
{
    __shared__ HashLds<NS, kMaxW> lds;
    const uint32_t lane = lane_id();
    const uint32_t v = blockIdx.x;
    uint64_t item;
    uint32_t lo, hi;  // the item's stream is searched for in [lo, hi)
    if (cm.n == 0) {  // every candidate of the call: wavefront v takes work item v
        item = v;
        if (item >= item_off[P * R]) return;
        lo = 0;
        hi = P * R;
    } else {
        if (v >= cm.wv0[cm.n]) return;
        uint32_t ci = 0;  // the last i with wv0[i] <= v
        {
            uint32_t h = cm.n;
            while (h - ci > 1) {
                const uint32_t mid = (ci + h) >> 1;
                if (cm.wv0[mid] <= v) ci = mid;
                else h = mid;
            }
        }
        const uint32_t cc = cm.cand[ci];
        item = (uint64_t)item_off[cc * R] + (v - cm.wv0[ci]);
        if (item >= item_off[(cc + 1) * R]) return;
        lo = cc * R;
        hi = (cc + 1) * R;
    }
    if (kSeq && !item_marked(aborted, item)) return;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (item_off[mid] <= item) lo = mid;
        else hi = mid;
    }
    const uint32_t c = lo / R;
    // kSeq: only the first marked segment of a run, which is never a stream's first item
    if (kSeq && (item == item_off[lo] || item_marked(aborted, item - 1))) return;
    const uint32_t d = lo - c * R;
    const uint32_t W = wa.W[c];
    if (W < (uint32_t)kMinW || W > (uint32_t)kMaxW) return;
    if (!kSeq && wa.grp[c] > 1u) return;  // k_replay_grp's segments (its marked ones come here in kSeq)
    static_assert(kList ? kMaxW < 64 : kMinW >= 64, "a list fits a register; a key repeated within 64 records always hits");
    const uint32_t* go = grp_off + (uint64_t)c * (R + 1u);
    const uint32_t gs = go[d], cnt = go[d + 1] - gs;
    const uint32_t S = seg_len(W, wa, wa.grp[c]);
    const uint32_t nseg = item_off[lo + 1] - item_off[lo];
    // [s0, s1): the records this wavefront replays; [s0, sc) of them are replayed only to
    // reach the state at sc (the run's predecessor in the kSeq pass)
    uint64_t i0 = item, i1 = item + 1;
    if (kSeq) {
        i0 = item - 1;
        while (i1 < item_off[lo + 1] && item_marked(aborted, i1)) ++i1;
    }
    const uint32_t s0 = seg_start((uint32_t)(i0 - item_off[lo]), nseg, cnt);
    const uint32_t sc = kSeq ? seg_start((uint32_t)(item - item_off[lo]), nseg, cnt) : s0;
    const uint32_t s1 = seg_start((uint32_t)(i1 - item_off[lo]), nseg, cnt);
    const uint64_t* __restrict__ rl = rec + (uint64_t)c * n + gs;
    if (!kSeq && lane == 0) aborted[item] = 0u;

    // State before record s0: the most recent W distinct keys of the records before it, then
    // those of the carried state. (A kSeq wavefront rebuilds an unmarked segment: in budget.)
    HashCache<NS, kMaxW> cache(lds, W, lane);
    cache.clear();
    uint32_t q = 0;
    if (!cache.rebuild(rl, s0, K, kSeq ? 0xFFFFFFFFu : rebuild_budget(S), q)) {
        if (lane == 0) aborted[item] = 1u;  // too few distinct keys in reach: left to the kSeq pass
        return;
    }
    if (q < W && lru_in) cache.rebuild_carried(lru_in + ((uint64_t)c * R + d) * max_W, K, q);
    q = q < W ? q : W;
    uint32_t skey = CR_EMPTY_SLOT;                 // kList: lane i = i-th most recent key
    const uint64_t wmask = (1ull << (W & 63u)) - 1ull;  // kList: lanes whose position is < W
    if (kList) skey = lane < q ? *cache.at(lds.list[lane]) : CR_EMPTY_SLOT;
    else cache.place(q);

    StreamStats st{stats, P, R, J, c, d, lane};
    bool bad = false;
    // Replay of records [r0, r1); the next batch of records is in flight while one is
    // replayed. With `on` false the cache advances but nothing is counted.
    auto run = [&](uint32_t r0, uint32_t r1, bool on) {
        uint64_t rv_next = r0 + lane < r1 ? rl[r0 + lane] : 0ull;
        for (uint32_t b0 = r0; b0 < r1; b0 += 64) {
            const uint32_t nb = r1 - b0 < 64u ? r1 - b0 : 64u;
            const uint64_t rv = rv_next;
            rv_next = b0 + 64u + lane < r1 ? rl[b0 + 64u + lane] : 0ull;
            const uint32_t kl = lane < nb ? (uint32_t)rv : CR_EMPTY_SLOT;
            const bool vl = lane < nb && kl < K;
            bad |= lane < nb && kl >= K;
            const uint32_t pl = vl && on ? prefix_len[kl] : 0u;  // consumed after the batch
            const uint64_t vm = ballot(vl);
            uint64_t hm;  // the lanes whose records hit
            if (!kList) {
                hm = cache.step(kl, vm);
            } else {
                uint32_t depth = 0xFFFFFFFFu;  // lane t: hit depth of record t
                if (vm == ~0ull) {
                    depth = mtf_batch(skey, rl + b0, wmask);
                } else {
                    for (uint32_t t = 0; t < nb; ++t) {
                        const uint32_t kk = rdlane(kl, t);
                        if (kk < K) depth = wrlane(depth, mtf_step(skey, kk, wmask), t);
                    }
                }
                hm = ballot(depth != 0xFFFFFFFFu);
            }
            if (on) st.add(rv, vm, hm, pl);
        }
        st.flush();
    };
    if (sc > s0) run(s0, sc < s1 ? sc : s1, false);
    run(sc, s1, true);
    if (ballot(bad) && lane == 0) atomicOr(err, CR_ERR_KEY_RANGE);
    if (s1 == cnt) {
        uint32_t* __restrict__ lo_ = lru_out + ((uint64_t)c * R + d) * max_W;
        if (kList) {
            for (uint32_t idx = lane; idx < max_W; idx += 64) lo_[idx] = idx < W ? skey : CR_EMPTY_SLOT;
        } else {
            cache.each_live([&](uint32_t key, uint32_t depth) { lo_[depth] = key; });
            for (uint32_t idx = cache.live + lane; idx < max_W; idx += 64) lo_[idx] = CR_EMPTY_SLOT;
        }
    }
}

// ---------------------------------------------------------------------------------------
// Small lists, several segments per wavefront (calls with one interval). A list of
// W <= 64 / G slots needs W lanes, so a wavefront keeps G lists side by side in lane groups
// of w = 64 / G lanes (group g: lanes g w .. g w + w - 1, position j in lane g w + j), each
// replaying its own segment, and one instruction advances all G of them. Per step, group g
// reads its record's key from LDS into all of its lanes; one compare gives the hit mask m
// (at most one lane per group). With END the lanes of position W - 1 and START those of
// position 0, M = m | END has a set bit in every group and its lowest one at or above the
// group's START is the hit (or position W - 1 on a miss), so the borrow of M - START runs
// exactly over positions 0 .. hit of each group: M ^ (M - START) is the set of lanes that
// move back by one, in every group at once. The move is one select with a wave_shr:1 DPP
// source, and the key goes into each group's position 0 by a second select. Groups without
// a record at a step (segment ended, key out of range) read a marker key that matches no
// slot and are masked out of both selects.
//
// The state before a segment is rebuilt forward: the D records before it are replayed from
// an empty list (from the carried state where the window reaches the stream start). When
// the window holds W distinct keys the list is exactly the W most recent ones, so it is full
// when it is right; otherwise D grows, up to kGrpRebuildBudget S rounded up to whole
// 64-record batches. A segment whose window still holds fewer than W distinct keys there is
// marked in `aborted`, and the kSeq pass of k_replay replays it from its predecessor.
//
// Statistics: a step's hit is the bit of the lane that held its key; each lane shifts its
// bits into a register, and after a round of 64 steps the group's registers, OR-ed, give the
// round's hits. Every lane then adds the count, suffix + prefix lengths and the prefix
// lengths of the hits over the records it staged; the group's lanes are summed at the end.
constexpr uint32_t kGrpSent = 0xFFFFFFFEu;  // staged key of a skipped step: never a key (K <= 0xFFFFFFFE), never empty

// Positions 0 .. hit of every group move back by one: lanes with `keep` set hold their key,
// the others take their left neighbour's (a wave_shr:1 DPP source). The destination is the
// source, so lane 0, which has no left neighbour, keeps its key.
__device__ __forceinline__ void grp_move(uint32_t& sk, uint64_t movebits, uint64_t act)
{
    asm("s_nand_b64 vcc, %1, %2\n\t"
        "v_cndmask_b32_dpp %0, %0, %0, vcc wave_shr:1 row_mask:0xf bank_mask:0xf"
        : "+v"(sk)
        : "s"(movebits), "s"(act)
        : "vcc");
}

// h = 2 h + (this lane's bit of m): one add with carry-in
__device__ __forceinline__ void shift_in_lane_bit(uint32_t& h, uint64_t m)
{
    uint64_t dummy;
    asm("v_addc_co_u32 %0, %1, %0, %0, %2" : "+v"(h), "=s"(dummy) : "s"(m));
}

template <int G>
__global__ __launch_bounds__(kReplayThreads) void k_replay_grp(
    const uint64_t* __restrict__ rec, uint64_t n, const uint32_t* __restrict__ grp_off,
    const uint32_t* __restrict__ item_off, const uint32_t* __restrict__ gwave_off, uint32_t P, uint32_t R, uint32_t K,
    const uint32_t* __restrict__ prefix_len, WArg wa, uint32_t max_W, const uint32_t* __restrict__ lru_in,
    uint32_t* __restrict__ lru_out, uint64_t* __restrict__ stats, uint8_t* __restrict__ aborted,
    uint32_t* __restrict__ err)
{
    constexpr uint32_t w = 64u / G;
    constexpr uint32_t kStride = 65u;  // keys per group in the stage (padded: groups on other banks)
    __shared__ uint32_t s_stage[kReplayThreads / 64][G * kStride];
    const uint32_t lane = lane_id(), wv = wave_in_block();
    const uint32_t g = lane / w, j = lane % w;
    const uint32_t wid = blockIdx.x * (kReplayThreads / 64u) + wv;
    if (wid >= gwave_off[P]) return;
    uint32_t c = 0;  // the candidate: the last c with gwave_off[c] <= wid
    {
        uint32_t hi = P;
        while (hi - c > 1) {
            const uint32_t mid = (c + hi) >> 1;
            if (gwave_off[mid] <= wid) c = mid;
            else hi = mid;
        }
    }
    if (wa.grp[c] != (uint32_t)G) return;
    const uint32_t W = wa.W[c];
    const uint64_t it1 = item_off[(uint64_t)(c + 1) * R];
    const uint64_t item = item_off[(uint64_t)c * R] + (uint64_t)G * (wid - gwave_off[c]) + g;
    bool live = item < it1;
    uint32_t lo = c * R;  // the item's stream
    if (live) {
        uint32_t hi = (c + 1) * R;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (item_off[mid] <= item) lo = mid;
            else hi = mid;
        }
    }
    const uint32_t d = lo - c * R;
    const uint32_t S = seg_len(W, wa, G);
    const uint32_t* go = grp_off + (uint64_t)c * (R + 1u);
    const uint32_t gs = live ? go[d] : 0u, cnt = live ? go[d + 1] - gs : 0u;
    const uint32_t nseg = live ? item_off[lo + 1] - item_off[lo] : 1u;
    const uint32_t s0 = live ? seg_start((uint32_t)(item - item_off[lo]), nseg, cnt) : 0u;
    const uint32_t s1 = live ? seg_start((uint32_t)(item - item_off[lo]) + 1u, nseg, cnt) : 0u;
    const uint64_t* __restrict__ rl = rec + (uint64_t)c * n + gs;
    if (live && j == 0) aborted[item] = 0u;
    uint32_t* __restrict__ stage = s_stage[wv] + g * kStride;

    uint64_t START = 0, END = 0;
#pragma unroll
    for (uint32_t q = 0; q < G; ++q) {
        START |= 1ull << (q * w);
        END |= 1ull << (q * w + W - 1u);
    }
    uint32_t sk = CR_EMPTY_SLOT;
    bool bad = false;
    uint32_t a_hit = 0, a_req = 0;
    uint64_t a_hp = 0, a_all = 0;

    // One step of every group: key kv (kGrpSent: none). With hb, each lane shifts its hit
    // bit of the step into hb (hb = 2 hb + hit: after 32 steps, step t is bit 31 - t).
    auto step = [&](uint32_t kv, uint32_t* hb) {
        const uint64_t m = ballot(sk == kv);
        const uint64_t act = ballot(kv != kGrpSent);
        const uint64_t M = m | END;
        grp_move(sk, M ^ (M - START), act);
        sk = __builtin_amdgcn_inverse_ballot_w64(START & act) ? kv : sk;
        if (hb) shift_in_lane_bit(*hb, m);
    };
    // Records [a, a + len) of each group's stream through its list, in rounds of 64 steps:
    // lane j of a group stages the keys of steps j, j + w, ... of its group in LDS. The next
    // round's records are loaded while a round runs. With statistics, the prefix lengths of
    // a round's records are gathered as it starts and used once it has run: every round is
    // 64 steps (idle ones at the end of a group's range), and the hit bits of the group's
    // lanes, OR-ed together, say which of its steps hit.
    auto run = [&](uint32_t a, uint32_t len, bool with_stats) {
        uint32_t most = len;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const uint32_t x = __shfl_xor(most, o, 64);
            most = x > most ? x : most;
        }
        most = __builtin_amdgcn_readfirstlane(most);
        uint64_t rv[G];
#pragma unroll
        for (uint32_t i = 0; i < G; ++i) {
            const uint32_t t = j + w * i;
            rv[i] = t < len ? rl[a + t] : 0ull;
        }
        for (uint32_t t0 = 0; t0 < most; t0 += 64u) {
            uint32_t key[G], sfx[G];
            bool ok[G];
#pragma unroll
            for (uint32_t i = 0; i < G; ++i) {
                const uint32_t t = t0 + j + w * i;
                key[i] = (uint32_t)rv[i];
                sfx[i] = (uint32_t)(rv[i] >> 32) & 0xFFFFu;
                ok[i] = t < len && key[i] < K;
                bad |= t < len && key[i] >= K;
                stage[j + w * i] = ok[i] ? key[i] : kGrpSent;
            }
            uint32_t pl[G];
            if (with_stats) {
#pragma unroll
                for (uint32_t i = 0; i < G; ++i) pl[i] = prefix_len[ok[i] ? key[i] : 0u];
            }
#pragma unroll
            for (uint32_t i = 0; i < G; ++i) {  // the next round's records
                const uint32_t t = t0 + 64u + j + w * i;
                rv[i] = t < len ? rl[a + t] : 0ull;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (with_stats) {
                uint32_t h0 = 0, h1 = 0;
#pragma unroll
                for (uint32_t t = 0; t < 32u; ++t) step(stage[t], &h0);
#pragma unroll
                for (uint32_t t = 32; t < 64u; ++t) step(stage[t], &h1);
#pragma unroll
                for (uint32_t o = w / 2; o >= 1; o >>= 1) {
                    h0 |= __shfl_xor(h0, o, 64);
                    h1 |= __shfl_xor(h1, o, 64);
                }
                if (j == 0) a_hit += __builtin_popcount(h0) + __builtin_popcount(h1);
#pragma unroll
                for (uint32_t i = 0; i < G; ++i) {
                    const uint32_t t = j + w * i;
                    const bool hit = ((t < 32u ? h0 >> (31u - t) : h1 >> (63u - t)) & 1u) != 0u;
                    a_req += ok[i] ? 1u : 0u;
                    a_all += ok[i] ? (uint64_t)sfx[i] + pl[i] : 0ull;
                    a_hp += ok[i] && hit ? (uint64_t)pl[i] : 0ull;
                }
            } else {
                const uint32_t nt = most - t0 < 64u ? most - t0 : 64u;
                if (nt == 64u) {
#pragma unroll 16
                    for (uint32_t t = 0; t < 64u; ++t) step(stage[t], nullptr);
                } else {
                    for (uint32_t t = 0; t < nt; ++t) step(stage[t], nullptr);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    };
    // The carried state of the groups in `on`, oldest entry first, through their lists: the
    // entries before the row's first empty slot, keys >= K skipped, as the backward rebuild
    // appends them.
    auto carried = [&](bool on) {
        const uint32_t* __restrict__ li = lru_in + ((uint64_t)c * R + d) * max_W;
        const uint32_t v = on && j < W ? li[j] : CR_EMPTY_SLOT;
        uint32_t fe = W;  // the row's first empty slot
        for (uint32_t i = 0; i < W; ++i) {
            const uint32_t x = __shfl(v, g * w + i, 64);
            fe = x == CR_EMPTY_SLOT && fe == W ? i : fe;
        }
        for (uint32_t i = W; i-- > 0;) {
            const uint32_t x = __shfl(v, g * w + i, 64);
            step(on && i < fe && x < K ? x : kGrpSent, nullptr);
        }
    };

    // rebuild the state at s0
    const uint32_t budget = (kGrpRebuildBudget * S + 63u) & ~63u;
    const uint32_t dmax = s0 < budget ? s0 : budget;
    bool ready = !live || s0 == 0;
    if (lru_in && ballot(live && s0 == 0)) carried(live && s0 == 0);
    for (uint32_t D = 4u * W; ballot(!ready) != 0; D *= 8u) {
        const bool part = !ready;
        const uint32_t dg = D < dmax ? D : dmax;
        sk = part ? CR_EMPTY_SLOT : sk;
        if (lru_in && ballot(part && dg == s0)) carried(part && dg == s0);
        run(s0 - dg, part ? dg : 0u, false);
        const uint64_t F = ballot(j == W - 1u && sk != CR_EMPTY_SLOT);
        const bool full = (F >> (g * w + W - 1u)) & 1ull;
        const bool ok = part && (full || dg == s0);
        if (part && !ok && dg == dmax) {  // too few distinct keys in reach: left to the kSeq pass
            if (j == 0) aborted[item] = 1u;
            live = false;
        }
        ready = ready || ok || (part && dg == dmax);
    }
    run(s0, live ? s1 - s0 : 0u, true);
    if (ballot(bad) && lane == 0) atomicOr(err, CR_ERR_KEY_RANGE);
    // the group's sums in its lane 0
#pragma unroll
    for (uint32_t o = w / 2; o >= 1; o >>= 1) {
        a_hit += __shfl_xor(a_hit, o, 64);
        a_req += __shfl_xor(a_req, o, 64);
        a_hp += (uint64_t)__shfl_xor((unsigned long long)a_hp, o, 64);
        a_all += (uint64_t)__shfl_xor((unsigned long long)a_all, o, 64);
    }
    if (live && j == 0) {
        unsigned long long* st = (unsigned long long*)(stats + ((uint64_t)c * R + d) * 4u);  // interval 0
        atomicAdd(st + 0, (unsigned long long)a_req);
        if (a_hit) atomicAdd(st + 1, (unsigned long long)a_hit);
        atomicAdd(st + 2, (unsigned long long)(a_all - a_hp));
        if (a_hp) atomicAdd(st + 3, (unsigned long long)a_hp);
    }
    if (live && s1 == cnt) {
        uint32_t* __restrict__ lo_ = lru_out + ((uint64_t)c * R + d) * max_W;
        if (j < W) lo_[j] = sk;
        for (uint32_t idx = W + j; idx < max_W; idx += w) lo_[idx] = CR_EMPTY_SLOT;
    }
}

struct ReplayArgs {
    WArg wa;
    uint32_t classes;    // bit rep_class: some candidate's list is of that class
    uint32_t wclasses;   // the same, candidates replayed one list per wavefront only
    uint32_t groups;     // bit G: some candidate is replayed by k_replay_grp<G>
    uint64_t grp_waves;  // bound on k_replay_grp wavefronts
};

// Records (n times the number of candidates with W <= 16) from which a one-interval call
// replays those candidates by k_replay_grp; below it there are too few segments to fill the
// chip with a G-th of the wavefronts.
uint64_t g_grp_min_records = 1ull << 25;

inline cr_status replay_args(uint64_t n, uint32_t J, uint32_t P, uint32_t R, const uint32_t* W, uint32_t max_W,
                             size_t ws_bytes, void* ws, ReplayArgs* ra)
{
    if (P == 0 || P > CR_MAX_CANDS || R == 0 || R > CR_MAX_R || J == 0 || J > CR_MAX_J || !W || max_W == 0 ||
        max_W > CR_MAX_W || !ws || n >= 0xFFFFFFFFull)
        return CR_EINVAL;
    ra->wa = WArg{};
    seg_rule(n, P, &ra->wa);
    ra->classes = 0;
    ra->wclasses = 0;
    ra->groups = 0;
    ra->grp_waves = 0;
    uint64_t small = 0;  // candidates k_replay_grp could take
    for (uint32_t c = 0; c < P; ++c) small += grp_of(W[c], J) > 1u ? 1u : 0u;
    const bool grouped = small > 0 && n * small >= g_grp_min_records;
    for (uint32_t c = 0; c < P; ++c) {
        if (W[c] == 0 || W[c] > max_W) return CR_EINVAL;
        ra->wa.W[c] = (uint16_t)W[c];
        const uint32_t G = grouped ? grp_of(W[c], J) : 1u;
        ra->wa.grp[c] = (uint8_t)G;
        ra->classes |= 1u << rep_class(W[c]);
        if (G == 1u) ra->wclasses |= 1u << rep_class(W[c]);
        const uint32_t S = seg_len(W[c], ra->wa, G);
        if (G > 1u) {  // at most R + n / S work items, G per wavefront
            ra->groups |= 1u << G;
            ra->grp_waves += ((uint64_t)R + n / S) / G + 1u;
        }
    }
    if (ws_bytes < replay_layout(nullptr, n, P, R).bytes) return CR_ESIZE;
    return CR_OK;
}

inline void* ws_base(void* ws) { return reinterpret_cast<void*>(((uintptr_t)ws + 255) & ~(uintptr_t)255); }

}  // namespace
}  // namespace cr

extern "C" void cr_replay_set_group_min_records(uint64_t min_records) { cr::g_grp_min_records = min_records; }

extern "C" size_t cr_replay_workspace_bytes(uint64_t n, uint32_t P, uint32_t R)
{
    return cr::replay_layout(nullptr, n, P, R).bytes;
}

extern "C" size_t cr_workspace_bytes(uint32_t num_keys, uint32_t R, uint32_t P, uint64_t max_n)
{
    const size_t a = cr_count_slice_workspace_bytes(max_n, num_keys), b = cr_replay_workspace_bytes(max_n, P, R);
    return a > b ? a : b;
}

extern "C" size_t cr_lru_state_bytes(uint32_t P, uint32_t R, uint32_t max_W)
{
    return (size_t)P * R * max_W * sizeof(uint32_t);
}

namespace cr {
namespace {
__global__ void k_lru_fill(uint32_t* __restrict__ p, uint64_t n)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = CR_EMPTY_SLOT;
}
}  // namespace
}  // namespace cr

extern "C" cr_status cr_lru_reset(uint32_t* lru_state, uint32_t P, uint32_t R, uint32_t max_W, void* stream)
{
    using namespace cr;
    if (!lru_state || P == 0 || P > CR_MAX_CANDS || R == 0 || R > CR_MAX_R || max_W == 0 || max_W > CR_MAX_W)
        return CR_EINVAL;
    const uint64_t n = (uint64_t)P * R * max_W;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_lru_fill, dim3((uint32_t)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096)), dim3(256), 0,
                       as_stream(stream), lru_state, n);
    return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
}

extern "C" cr_status cr_replay_partition(const uint32_t* keys, const uint16_t* suffix, const uint16_t* dest,
                                         uint64_t n, const uint64_t* off, uint32_t J, uint32_t P, uint32_t R,
                                         const uint32_t* W, void* ws, size_t ws_bytes, uint32_t* err, void* stream)
{
    using namespace cr;
    ReplayArgs ra;
    uint32_t mw = 0;
    for (uint32_t c = 0; W && c < P && c < CR_MAX_CANDS; ++c) mw = W[c] > mw ? W[c] : mw;
    const cr_status v = replay_args(n, J, P, R, W, mw ? mw : 1u, ws_bytes, ws, &ra);
    if (v != CR_OK) return v;
    if (!off || !err || (n > 0 && (!keys || !suffix || !dest))) return CR_EINVAL;
    const ReplayWs w = replay_layout(ws_base(ws), n, P, R);
    PartGeom g = part_geom(n, P);
    // R > 64: whole sub-tiles of the wide scatter, however few (a tile of 1,024 occupies one
    // wavefront of a block, whose phases are as long as a full sub-tile's: 4,000,037 x 4 candidates, 257
    // destinations 210 -> 81 us; 1e6 x 1, 65 destinations 57 -> 31 us; 1e5 x 1 31 -> 29 us)
    const bool one = J == 1 && P * ((n + 8191u) / 8192u) >= kWideMinBlocks;
    if (R > 64) {
        const uint64_t sub = 1024u * (one ? wide_waves<true>() : wide_waves<false>());
        g.tile = (g.tile + sub - 1) / sub * sub;
        g.ntiles = (n + g.tile - 1) / g.tile;
    }
    const hipStream_t st = as_stream(stream);
    (void)hipGetLastError();
    // 16-byte loads of keys, destinations and suffixes need 16-byte aligned rows
    const bool vec = ((uintptr_t)keys & 15u) == 0 && ((uintptr_t)suffix & 15u) == 0 && ((uintptr_t)dest & 15u) == 0 &&
                     (n & 7u) == 0;
    if (g.ntiles && vec)
        hipLaunchKernelGGL(k_part_hist<true>, dim3((uint32_t)g.ntiles, P), dim3(kHistThreads), (size_t)R * 4u, st, dest,
                           n, R, g.tile, g.ntiles, w.tcnt, err);
    else if (g.ntiles)
        hipLaunchKernelGGL(k_part_hist<false>, dim3((uint32_t)g.ntiles, P), dim3(kHistThreads), (size_t)R * 4u, st, dest,
                           n, R, g.tile, g.ntiles, w.tcnt, err);
    hipLaunchKernelGGL(k_scan_dest, dim3(R, P), dim3(kScanThreads), 0, st, w.tcnt, g.ntiles, R, w.dtot);
    hipLaunchKernelGGL(k_seg_items, dim3(1), dim3(1024), 0, st, w.dtot, P, R, ra.wa, w.grp_off, w.item_off,
                       w.gwave_off);
    if (g.ntiles && R <= 64 && vec)
        hipLaunchKernelGGL(k_part_scatter64<true>, dim3(P * xcd_grid((uint32_t)g.ntiles)), dim3(64),
                           kScatter64Lds, st, keys, suffix, dest, n, off, J, P, R, g.tile, g.ntiles, w.tcnt,
                           w.grp_off, w.rec);
    else if (g.ntiles && R <= 64)
        hipLaunchKernelGGL(k_part_scatter64<false>, dim3(P * xcd_grid((uint32_t)g.ntiles)), dim3(64),
                           kScatter64Lds, st, keys, suffix, dest, n, off, J, P, R, g.tile, g.ntiles, w.tcnt,
                           w.grp_off, w.rec);
    else if (g.ntiles) {
#define CR_WIDE(ONE)                                                                                                \
    do {                                                                                                            \
        const size_t lds = scatter_wide_lds_bytes<ONE>(R);                                                          \
        if (hipFuncSetAttribute((const void*)k_part_scatter_wide<ONE>, hipFuncAttributeMaxDynamicSharedMemorySize,   \
                                (int)lds) != hipSuccess)                                                            \
            return CR_EHIP;                                                                                         \
        hipLaunchKernelGGL(k_part_scatter_wide<ONE>, dim3(P * xcd_grid((uint32_t)g.ntiles)), dim3(64u * wide_waves<ONE>()), lds, \
                           st, keys, suffix, dest, n, off, J, P, R, g.tile, g.ntiles, w.tcnt, w.grp_off,       \
                           w.rec);                                                                                  \
    } while (0)
        if (one) CR_WIDE(true);
        else CR_WIDE(false);
#undef CR_WIDE
    }
    return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
}

namespace cr {
namespace {
// Two side streams per device (default priority) for the list-size launches of a replay
// call, created on a device's first call and kept until the process ends. A launch runs as
// many wavefronts as its segments, and near its end the chip empties while its last
// segments finish; on two streams one list size's launch fills the room another's leaves.
// The calls that share them are serialised by a host mutex (fork, launches and join).
#ifndef CR_REPLAY_SIDE_STREAMS
#define CR_REPLAY_SIDE_STREAMS 1
#endif
constexpr int kSideDevices = 64;
struct SideStreams {
    bool ready = false, failed = false;
    hipStream_t s[2] = {nullptr, nullptr};
    hipEvent_t fork = nullptr, join[2] = {nullptr, nullptr};
};
std::mutex g_side_mu;
SideStreams g_side[kSideDevices];

// The current device's side streams (caller holds g_side_mu), or nullptr: then the launches
// stay on the caller's stream. A device whose streams or events could not all be created
// releases what was made and is not tried again.
SideStreams* side_streams()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kSideDevices) return nullptr;
    SideStreams& q = g_side[dev];
    if (!q.ready && !q.failed) {
        bool ok = hipEventCreateWithFlags(&q.fork, hipEventDisableTiming) == hipSuccess;
        for (int i = 0; i < 2 && ok; ++i)
            ok = hipStreamCreateWithFlags(&q.s[i], hipStreamNonBlocking) == hipSuccess &&
                 hipEventCreateWithFlags(&q.join[i], hipEventDisableTiming) == hipSuccess;
        if (!ok) {
            for (int i = 0; i < 2; ++i) {
                if (q.join[i]) (void)hipEventDestroy(q.join[i]);
                if (q.s[i]) (void)hipStreamDestroy(q.s[i]);
                q.join[i] = nullptr;
                q.s[i] = nullptr;
            }
            if (q.fork) (void)hipEventDestroy(q.fork);
            q.fork = nullptr;
            (void)hipGetLastError();
            q.failed = true;
        }
        q.ready = ok;
    }
    return q.ready ? &q : nullptr;
}
}  // namespace
}  // namespace cr

extern "C" cr_status cr_replay_lru(const uint32_t* prefix_len, uint32_t num_keys, uint64_t n, uint32_t J,
                                   uint32_t P, uint32_t R, const uint32_t* W, uint32_t max_W, const uint32_t* lru_in,
                                   uint32_t* lru_out, uint64_t* stats, void* ws, size_t ws_bytes, uint32_t* err,
                                   void* stream)
{
    using namespace cr;
    ReplayArgs ra;
    const cr_status v = replay_args(n, J, P, R, W, max_W, ws_bytes, ws, &ra);
    if (v != CR_OK) return v;
    if (num_keys == 0 || num_keys == 0xFFFFFFFFu || !prefix_len || !lru_out || !stats || !err) return CR_EINVAL;
    if (lru_in && lru_in < lru_out + (uint64_t)P * R * max_W && lru_out < lru_in + (uint64_t)P * R * max_W)
        return CR_EINVAL;
    const ReplayWs w = replay_layout(ws_base(ws), n, P, R);
    const hipStream_t st = as_stream(stream);
    const uint64_t gblocks = (ra.grp_waves + (kReplayThreads / 64) - 1) / (kReplayThreads / 64);
    if (gblocks > 0x7FFFFFFFull) return CR_EINVAL;
    // One launch per list class, with wavefronts for its own candidates only: a stream of cnt
    // records has max(1, ceil(cnt / S)) work items, so a candidate has at most R + n / S of them.
    CandMap cm;
    auto cand_map = [&](uint32_t cls, bool seq) -> uint64_t {
        uint64_t wv = 0;
        cm.n = 0;
        for (uint32_t c = 0; c < P; ++c) {
            if (rep_class(W[c]) != cls || (!seq && ra.wa.grp[c] > 1u)) continue;
            cm.cand[cm.n] = (uint16_t)c;
            cm.wv0[cm.n++] = (uint32_t)wv;
            wv += (uint64_t)R + n / seg_len(W[c], ra.wa, ra.wa.grp[c]) + 1u;
        }
        cm.wv0[cm.n] = (uint32_t)wv;
        if (cm.n == P) cm.n = 0;  // every candidate, in order: work item v is wavefront v
        return wv;
    };
    for (uint32_t cls = 0; cls < kClasses; ++cls)
        if (cand_map(cls, true) > 0x7FFFFFFFull) return CR_EINVAL;
    (void)hipGetLastError();
    auto launch_class = [&](uint32_t cls, bool seq, hipStream_t on) {
        const uint64_t nw = cand_map(cls, seq);
        if (!nw) return;
#define CR_REPLAY(KERNEL)                                                                                            \
    hipLaunchKernelGGL(KERNEL, dim3((uint32_t)nw), dim3(64), 0, on, w.rec, n, w.grp_off, w.item_off, P, R, num_keys, \
                       J, prefix_len, ra.wa, cm, max_W, lru_in, lru_out, stats, w.aborted, err)
#define CR_CLASS(C, LIST)                                                                                            \
    if (cls == (C)) {                                                                                               \
        if (seq) CR_REPLAY((k_replay<kSlots[C], (C) ? kMaxW[(C) - 1] + 1 : 1, kMaxW[C], LIST, true>));               \
        else CR_REPLAY((k_replay<kSlots[C], (C) ? kMaxW[(C) - 1] + 1 : 1, kMaxW[C], LIST, false>));                  \
    }
        CR_CLASS(0, true) CR_CLASS(1, false) CR_CLASS(2, false) CR_CLASS(3, false) CR_CLASS(4, false)
#undef CR_CLASS
#undef CR_REPLAY
    };
    // The list classes' launches and the grouped ones are independent of each other (other
    // candidates; every work item has a mark of its own); the kSeq passes read what all
    // of them marked, so they follow on the caller's stream after the join. A call under
    // stream capture keeps everything on the caller's stream.
    uint32_t nlaunch = __builtin_popcount(ra.wclasses) + __builtin_popcount(ra.groups);
    std::unique_lock<std::mutex> side_lock;
    SideStreams* side = nullptr;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (CR_REPLAY_SIDE_STREAMS && nlaunch >= 2 && hipStreamIsCapturing(st, &cap) == hipSuccess &&
        cap == hipStreamCaptureStatusNone) {
        side_lock = std::unique_lock<std::mutex>(g_side_mu);
        side = side_streams();
    }
    hipStream_t lane_st[2] = {st, st};
    if (side) {
        if (hipEventRecord(side->fork, st) != hipSuccess || hipStreamWaitEvent(side->s[0], side->fork, 0) != hipSuccess ||
            hipStreamWaitEvent(side->s[1], side->fork, 0) != hipSuccess)
            return CR_EHIP;
        lane_st[0] = side->s[0];
        lane_st[1] = side->s[1];
    }
    // Launches in order of their work, each onto the stream with less work so far. A
    // launch's work is its candidates times a cost per candidate and request by list form,
    // in hundredths of the one-register list's (as measured alone: 0.47, 0.34, 0.35, 0.39 and
    // 0.44 ms per candidate and 4e7 requests; lists of 8 and 16 slots, replayed 8 and 4 per
    // wavefront, 0.56 and 0.77 of the one-register list).
    static constexpr uint32_t kCost[kClasses] = {100u, 71u, 74u, 82u, 93u};
    struct Launch { uint32_t kind; uint64_t work; };  // kind < kClasses: that class; 100 + G: k_replay_grp<G>
    Launch todo[kClasses + 2];
    uint32_t nt = 0;
    for (uint32_t cls = 0; cls < kClasses; ++cls)
        if (ra.wclasses & (1u << cls)) {
            uint64_t wk = 0;
            for (uint32_t c = 0; c < P; ++c)
                if (rep_class(W[c]) == cls && ra.wa.grp[c] == 1u) wk += kCost[cls];
            todo[nt++] = Launch{cls, wk};
        }
    for (uint32_t G = 4; G <= 8; G += 4)
        if (ra.groups & (1u << G)) {
            uint64_t wk = 0;
            for (uint32_t c = 0; c < P; ++c)
                if (ra.wa.grp[c] == G) wk += G == 8u ? 56u : 77u;
            todo[nt++] = Launch{100u + G, wk};
        }
    for (uint32_t a = 1; a < nt; ++a)  // insertion sort, heaviest first
        for (uint32_t b = a; b > 0 && todo[b].work > todo[b - 1].work; --b) {
            const Launch t = todo[b];
            todo[b] = todo[b - 1];
            todo[b - 1] = t;
        }
    uint64_t load[2] = {0, 0};
    for (uint32_t t = 0; t < nt; ++t) {
        const int li = load[1] < load[0] ? 1 : 0;  // the less loaded stream
        load[li] += todo[t].work;
        const hipStream_t ls = lane_st[li];
        const uint32_t k = todo[t].kind;
        if (k < kClasses) launch_class(k, false, ls);
        // several lists per wavefront; their marked segments join the kSeq pass of k_replay
#define CR_GRP(G)                                                                                                  \
        if (k == 100u + (G))                                                                                       \
            hipLaunchKernelGGL((k_replay_grp<G>), dim3((uint32_t)gblocks), dim3(kReplayThreads), 0, ls, w.rec, n,   \
                               w.grp_off, w.item_off, w.gwave_off, P, R, num_keys, prefix_len, ra.wa, max_W, lru_in, \
                               lru_out, stats, w.aborted, err);
        CR_GRP(4) CR_GRP(8)
#undef CR_GRP
    }
    if (side) {
        for (int i = 0; i < 2; ++i)
            if (hipEventRecord(side->join[i], side->s[i]) != hipSuccess ||
                hipStreamWaitEvent(st, side->join[i], 0) != hipSuccess)
                return CR_EHIP;
        side_lock.unlock();
    }
    for (uint32_t cls = 0; cls < kClasses; ++cls)
        if (ra.classes & (1u << cls)) launch_class(cls, true, st);
    return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
}

extern "C" cr_status cr_replay(const uint32_t* keys, const uint16_t* suffix, const uint32_t* prefix_len,
                               uint32_t num_keys, const uint16_t* dest, uint64_t n, const uint64_t* off, uint32_t J,
                               uint32_t P, uint32_t R, const uint32_t* W, uint32_t max_W, const uint32_t* lru_in,
                               uint32_t* lru_out, uint64_t* stats, void* ws, size_t ws_bytes, uint32_t* err,
                               void* stream)
{
    using namespace cr;
    ReplayArgs ra;
    cr_status v = replay_args(n, J, P, R, W, max_W, ws_bytes, ws, &ra);
    if (v != CR_OK) return v;
    if (num_keys == 0 || num_keys == 0xFFFFFFFFu || !prefix_len || !lru_out || !stats || !err || !off ||
        (n > 0 && (!keys || !suffix || !dest)))
        return CR_EINVAL;
    if (lru_in && lru_in < lru_out + (uint64_t)P * R * max_W && lru_out < lru_in + (uint64_t)P * R * max_W)
        return CR_EINVAL;
    v = cr_replay_partition(keys, suffix, dest, n, off, J, P, R, W, ws, ws_bytes, err, stream);
    if (v != CR_OK) return v;
    return cr_replay_lru(prefix_len, num_keys, n, J, P, R, W, max_W, lru_in, lru_out, stats, ws, ws_bytes, err,
                         stream);
}
