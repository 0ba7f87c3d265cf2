// Plan build: top-rate admission (Eq. 1; Section 3.1 "Warm-set admission"; Algorithm 1)
// and LPT placement (Section 3.1 "Placement and dispatch"; Algorithm 1 placement loop).
//
// Admission is split in two so that every candidate plan built from the same window
// shares one sort:
//   k_sort_window  one block per window: radix-select the C_max-th largest count, compact
//                  the keys at or above it in key order, and stable-LSD-radix-sort them by
//                  count (descending), which yields (count desc, key asc) exactly;
//   k_admit_plan   one block per plan: k by Eq. 1 in exact integers, block prefix sum of
//                  k, and the longest prefix whose sum fits C = R * W.
// LPT is a dependency chain of sum(k) steps per plan, cut into exact batches of
// consecutive jobs: one wavefront per plan for R <= 64 (k_lpt_small), one block of up to
// 1,024 threads per plan above that (k_lpt_block).
// k_plan_churn compares pairs of built plans for the replanning study.
#include <math.h>

#include <mutex>
#include <utility>

#include "cr_common.h"

namespace cr {
namespace {

constexpr int kSortThreads = 1024;

__host__ __device__ __forceinline__ bool hash_placed(uint32_t variant)
{
    return variant == CR_PLAN_AFFINITY || variant == CR_PLAN_REPLICATED;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += (uint64_t)__shfl_xor((unsigned long long)v, o, 64);
    return v;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t u = __shfl_xor(v, o, 64);
        v = u > v ? u : v;
    }
    return v;
}

__device__ __forceinline__ uint32_t wave_exscan_u32(uint32_t v, uint32_t* total)
{
    const uint32_t x = wave_incl_scan_u32(v);
    *total = rdlane(x, 63);
    return x - v;
}

constexpr uint32_t kSortBlock = 1024;                // 16 wavefronts per window
constexpr uint32_t kSortNW = kSortBlock / 64;
constexpr uint32_t kSortLdsRowBytes = 96u * 1024u;  // rows up to this size are staged in LDS

// Loads counts[b] for b = base + 4*tid + {0..3} (zero past K), 16 bytes per thread when
// the row allows it.
__device__ __forceinline__ uint4 load4(const uint32_t* __restrict__ row, uint32_t K, uint32_t b, bool vec)
{
    if (vec && b + 3 < K) return *reinterpret_cast<const uint4*>(row + b);
    return make_uint4(b < K ? row[b] : 0u, b + 1 < K ? row[b + 1] : 0u, b + 2 < K ? row[b + 2] : 0u,
                      b + 3 < K ? row[b + 3] : 0u);
}

// One 1024-thread block per window. The window's nonzero keys are ordered by (count desc,
// key asc) and cut at C_max in three steps, each with O(1) block barriers:
//  1. one pass over the row: nnz, max, sum and a histogram of min(count, 255); the
//     C_max-th largest count t is read off the histogram unless it is >= 255, in which
//     case an MSB radix select over the row finds it;
//  2. ordered compaction: every wavefront owns a contiguous slice of the row, counts
//     what it keeps, takes its offset from the other wavefronts' totals, and writes its
//     keys in key order (keys equal to t are kept up to the number still needed);
//  3. stable LSD radix sort by (max - count) over the kept entries, 8 bits per pass, each
//     wavefront scattering a contiguous slice with ballot-ranked digits.
// When the row fits, step 1 also stages it in LDS and the later passes read it there.
template <bool kRowLds>
__global__ __launch_bounds__(kSortBlock) void k_sort_window(const uint32_t* __restrict__ counts, uint32_t K,
                                                            uint32_t Cmax, uint32_t* __restrict__ order,
                                                            uint32_t* __restrict__ order_count,
                                                            uint32_t* __restrict__ n_order,
                                                            uint64_t* __restrict__ row_sum, uint2* __restrict__ buf)
{
    extern __shared__ uint32_t s_row[];  // [K] when kRowLds
    __shared__ uint32_t s_hist[kSortNW][256];
    __shared__ uint32_t s_h256[256];
    __shared__ uint32_t s_w[kSortNW][4];
    __shared__ uint32_t s_nnz, s_max, s_t, s_take;
    __shared__ unsigned long long s_sum;
    const uint32_t w = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wv = wave_in_block();
    const uint32_t* __restrict__ grow = counts + (uint64_t)w * K;
    const bool vec = (((uintptr_t)grow) & 15u) == 0;
    const uint32_t* row = kRowLds ? s_row : grow;
    uint2* b0 = buf + (uint64_t)w * 2u * Cmax;
    uint2* b1 = b0 + Cmax;
    for (uint32_t d = tid; d < 256; d += kSortBlock) s_h256[d] = 0;
    if (tid == 0) {
        s_nnz = 0;
        s_max = 0;
        s_sum = 0;
    }
    __syncthreads();
    // 1. statistics and the clamped histogram
    {
        uint32_t nnz = 0, mx = 0;
        uint64_t sum = 0;
        for (uint32_t b = 4 * tid; b < K; b += 4 * kSortBlock * 2) {
            const uint4 q0 = load4(grow, K, b, vec), q1 = load4(grow, K, b + 4 * kSortBlock, vec);
            const uint32_t cs[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
            if (kRowLds) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (b + u < K) s_row[b + u] = cs[u];
                    if (b + 4 * kSortBlock + u < K) s_row[b + 4 * kSortBlock + u] = cs[4 + u];
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t c = cs[u];
                if (c) {
                    ++nnz;
                    mx = c > mx ? c : mx;
                    sum += c;
                    atomicAdd(&s_h256[c < 255u ? c : 255u], 1u);
                }
            }
        }
        nnz = rdlane(wave_incl_scan_u32(nnz), 63);
        mx = wave_max_u32(mx);
        sum = wave_sum_u64(sum);
        if (lane == 0) {
            atomicAdd(&s_nnz, nnz);
            atomicMax(&s_max, mx);
            atomicAdd(&s_sum, (unsigned long long)sum);
        }
    }
    __syncthreads();
    const uint32_t nnz = s_nnz, mx = s_max;
    const uint32_t M = nnz < Cmax ? nnz : Cmax;
    if (tid == 0) {
        n_order[w] = M;
        row_sum[w] = s_sum;
    }
    if (M == 0) return;
    // threshold from the clamped histogram (wave 0, four bins per lane from 255 down)
    if (wv == 0) {
        uint32_t h[4], hs = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            h[q] = s_h256[255u - 4u * lane - q];
            hs += h[q];
        }
        uint32_t tot;
        uint32_t above = wave_exscan_u32(hs, &tot);
        uint32_t sel = 0, need = 0;
        bool found = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!found && above < M && above + h[q] >= M) {
                sel = 255u - 4u * lane - q;
                need = M - above;
                found = true;
            }
            above += h[q];
        }
        const uint32_t fl = first_lane(ballot(found));
        if (lane == 0) {
            s_t = rdlane(sel, fl);
            s_take = rdlane(need, fl);
        }
    }
    __syncthreads();
    if (s_t == 255u) {
        // the threshold is at least 255: MSB radix select over the row (rare)
        uint32_t prefix = 0, pmask = 0, need = M;
        for (int shift = 24; shift >= 0; shift -= 8) {
            if ((mx >> shift) == 0) {
                pmask |= 0xFFu << shift;
                continue;
            }
            __syncthreads();
            for (uint32_t d = tid; d < 256; d += kSortBlock) s_h256[d] = 0;
            __syncthreads();
            for (uint32_t b = tid; b < K; b += kSortBlock) {
                const uint32_t c = row[b];
                if (c != 0 && (c & pmask) == prefix) atomicAdd(&s_h256[(c >> shift) & 255u], 1u);
            }
            __syncthreads();
            if (wv == 0) {
                uint32_t h[4], hs = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h[q] = s_h256[255u - 4u * lane - q];
                    hs += h[q];
                }
                uint32_t tot;
                uint32_t above = wave_exscan_u32(hs, &tot);
                uint32_t sel = 0, nn = 0;
                bool found = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (!found && above < need && above + h[q] >= need) {
                        sel = 255u - 4u * lane - q;
                        nn = need - above;
                        found = true;
                    }
                    above += h[q];
                }
                const uint32_t fl = first_lane(ballot(found));
                if (lane == 0) {
                    s_t = rdlane(sel, fl);
                    s_take = rdlane(nn, fl);
                }
            }
            __syncthreads();
            prefix |= s_t << shift;
            pmask |= 0xFFu << shift;
            need = s_take;
        }
        __syncthreads();
        if (tid == 0) {
            s_t = prefix;
            s_take = need;
        }
        __syncthreads();
    }
    const uint32_t t = s_t, take_eq = s_take;

    // 2. ordered compaction, one contiguous slice of the row per wavefront
    const uint32_t span = (((K + kSortNW - 1) / kSortNW) + 63u) & ~63u;
    const uint32_t lo = wv * span < K ? wv * span : K, hi = lo + span < K ? lo + span : K;
    {
        uint32_t gt = 0, eq = 0;
        for (uint32_t b = lo + lane; b < hi; b += 64) {
            const uint32_t c = row[b];
            gt += c > t;
            eq += c == t;
        }
        gt = rdlane(wave_incl_scan_u32(gt), 63);
        eq = rdlane(wave_incl_scan_u32(eq), 63);
        if (lane == 0) {
            s_w[wv][0] = gt;
            s_w[wv][1] = eq;
        }
    }
    __syncthreads();
    {
        uint32_t eq_before = 0, sel_before = 0;
        for (uint32_t q = 0; q < wv; ++q) {
            const uint32_t eqq = s_w[q][1];
            const uint32_t left = take_eq > eq_before ? take_eq - eq_before : 0u;
            sel_before += s_w[q][0] + (eqq < left ? eqq : left);
            eq_before += eqq;
        }
        uint32_t running = sel_before, eq_seen = eq_before;
        for (uint32_t base = lo; base < hi; base += 64) {
            const uint32_t b = base + lane;
            const uint32_t c = b < hi ? row[b] : 0u;
            const uint64_t meq = ballot(b < hi && c == t);
            const uint32_t eq_rank = (uint32_t)__popcll(meq & lanemask_lt());
            const bool sel = b < hi && (c > t || (c == t && eq_seen + eq_rank < take_eq));
            const uint64_t ms = ballot(sel);
            const uint32_t pos = running + (uint32_t)__popcll(ms & lanemask_lt());
            if (sel && pos < M) b0[pos] = make_uint2(c, b);
            running += (uint32_t)__popcll(ms);
            eq_seen += (uint32_t)__popcll(meq);
        }
    }
    __syncthreads();

    // 3. stable LSD radix sort by v = mx - count (ascending v = descending count)
    const uint32_t range = mx - t;
    const uint32_t bits = range ? 32u - (uint32_t)__clz(range) : 0u;
    const uint32_t passes = (bits + 7u) / 8u;
    const uint32_t espan = (((M + kSortNW - 1) / kSortNW) + 63u) & ~63u;
    const uint32_t elo = wv * espan < M ? wv * espan : M, ehi = elo + espan < M ? elo + espan : M;
    uint2* src = b0;
    uint2* dst = b1;
    for (uint32_t pass = 0; pass < passes; ++pass) {
        const uint32_t shift = 8u * pass;
        for (uint32_t d = lane; d < 256; d += 64) s_hist[wv][d] = 0;
        for (uint32_t e = elo + lane; e < ehi; e += 64) atomicAdd(&s_hist[wv][((mx - src[e].x) >> shift) & 255u], 1u);
        __syncthreads();
        if (wv == 0) {  // offsets in (digit, wavefront) order
            uint32_t h[4][kSortNW], hs = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (uint32_t x = 0; x < kSortNW; ++x) {
                    h[q][x] = s_hist[x][4u * lane + q];
                    hs += h[q][x];
                }
            uint32_t tot;
            uint32_t ex = wave_exscan_u32(hs, &tot);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (uint32_t x = 0; x < kSortNW; ++x) {
                    s_hist[x][4u * lane + q] = ex;
                    ex += h[q][x];
                }
        }
        __syncthreads();
        for (uint32_t e0 = elo; e0 < ehi; e0 += 64) {
            const uint32_t e = e0 + lane;
            const bool valid = e < ehi;
            const uint2 kv = valid ? src[e] : make_uint2(0u, 0u);
            const uint32_t d = valid ? ((mx - kv.x) >> shift) & 255u : 0u;
            uint64_t peers = ballot(valid);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool on = (d >> bit) & 1u;
                const uint64_t bb = ballot(on);
                peers &= on ? bb : ~bb;
            }
            const uint32_t rk = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t at = valid ? s_hist[wv][d] + rk : 0u;
            if (valid && at < M) dst[at] = kv;
            if (valid && rk == 0) atomicAdd(&s_hist[wv][d], (uint32_t)__popcll(peers));
        }
        __syncthreads();
        uint2* tmp = src;
        src = dst;
        dst = tmp;
    }
    uint32_t* __restrict__ ord = order + (uint64_t)w * Cmax;
    uint32_t* __restrict__ ocnt = order_count + (uint64_t)w * Cmax;
    for (uint32_t e = tid; e < M; e += kSortBlock) {
        const uint2 kv = src[e];
        ord[e] = kv.y;
        ocnt[e] = kv.x;
    }
}

// Register-resident variant for rows of up to 1024 * kNpl keys and C_max <= kRegCmax:
// wavefront wv keeps its contiguous slice of the row in registers (kNpl values per lane,
// all loads in flight together), so the row is read from memory once and no LDS row copy
// limits the blocks per CU; the kept entries and both radix buffers live in LDS. Counts
// 1..3, the bulk of a long-tailed row, are histogrammed by ballots instead of contended
// LDS atomics. Same three steps and results as k_sort_window.
constexpr uint32_t kRegCmax = 2048;

// Up to 20 counts per thread the kernel fits 64 VGPRs, which leaves room for two blocks
// per CU (8 wavefronts per SIMD); the windows are independent, so that halves the rounds.
template <int kNpl>
__global__ __launch_bounds__(kSortBlock, kNpl <= 20 ? 8 : 1) void k_sort_window_reg(const uint32_t* __restrict__ counts, uint32_t K,
                                                                uint32_t Cmax, uint32_t* __restrict__ order,
                                                                uint32_t* __restrict__ order_count,
                                                                uint32_t* __restrict__ n_order,
                                                                uint64_t* __restrict__ row_sum)
{
    __shared__ uint2 s_buf[2][kRegCmax];
    __shared__ uint32_t s_hist[kSortNW][256];
    __shared__ uint32_t s_h256[256];
    __shared__ uint32_t s_w[kSortNW][2];
    __shared__ uint32_t s_nnz, s_max, s_t, s_take;
    __shared__ unsigned long long s_sum;
    const uint32_t w = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wv = wave_in_block();
    const uint32_t* __restrict__ grow = counts + (uint64_t)w * K;
    const uint32_t span = (((K + kSortNW - 1) / kSortNW) + 63u) & ~63u;  // <= 64 * kNpl
    const uint32_t lo = wv * span < K ? wv * span : K, hi = lo + span < K ? lo + span : K;
    uint32_t v[kNpl];
    {  // the slice through a buffer resource: entries at or past hi read as 0
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(grow + lo, (hi - lo) * 4u);
#pragma unroll
        for (int i = 0; i < kNpl; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, (64u * i + lane) * 4u, 0, 0);
    }
    for (uint32_t d = tid; d < 256; d += kSortBlock) s_h256[d] = 0;
    if (tid == 0) {
        s_nnz = 0;
        s_max = 0;
        s_sum = 0;
    }
    __syncthreads();
    // 1. statistics and the clamped histogram
    {
        uint32_t nnz = 0, mx = 0, n1 = 0, n2 = 0, n3 = 0;  // per lane
        uint64_t sum = 0;
#pragma unroll
        for (int i = 0; i < kNpl; ++i) {
            const uint32_t c = v[i];
            nnz += c != 0u;
            n1 += c == 1u;
            n2 += c == 2u;
            n3 += c == 3u;
            mx = c > mx ? c : mx;
            sum += c;
            if (c >= 4u) atomicAdd(&s_h256[c < 255u ? c : 255u], 1u);
            __builtin_amdgcn_sched_barrier(0);
        }
        nnz = wave_sum_u32(nnz);
        n1 = wave_sum_u32(n1);
        n2 = wave_sum_u32(n2);
        n3 = wave_sum_u32(n3);
        mx = wave_max_u32(mx);
        sum = wave_sum_u64(sum);
        if (lane == 0) {
            atomicAdd(&s_nnz, nnz);
            atomicMax(&s_max, mx);
            atomicAdd(&s_sum, (unsigned long long)sum);
            if (n1) atomicAdd(&s_h256[1], n1);
            if (n2) atomicAdd(&s_h256[2], n2);
            if (n3) atomicAdd(&s_h256[3], n3);
        }
    }
    __syncthreads();
    const uint32_t nnz = s_nnz, mx = s_max;
    const uint32_t M = nnz < Cmax ? nnz : Cmax;
    if (tid == 0) {
        n_order[w] = M;
        row_sum[w] = s_sum;
    }
    if (M == 0) return;
    if (wv == 0) {  // threshold from the clamped histogram, four bins per lane from 255 down
        uint32_t h[4], hs = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            h[q] = s_h256[255u - 4u * lane - q];
            hs += h[q];
        }
        uint32_t tot;
        uint32_t above = wave_exscan_u32(hs, &tot);
        uint32_t sel = 0, need = 0;
        bool found = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!found && above < M && above + h[q] >= M) {
                sel = 255u - 4u * lane - q;
                need = M - above;
                found = true;
            }
            above += h[q];
        }
        const uint32_t fl = first_lane(ballot(found));
        if (lane == 0) {
            s_t = rdlane(sel, fl);
            s_take = rdlane(need, fl);
        }
    }
    __syncthreads();
    if (s_t == 255u) {  // the threshold is at least 255: MSB radix select over the registers
        uint32_t prefix = 0, pmask = 0, need = M;
        for (int shift = 24; shift >= 0; shift -= 8) {
            if ((mx >> shift) == 0) {
                pmask |= 0xFFu << shift;
                continue;
            }
            __syncthreads();
            for (uint32_t d = tid; d < 256; d += kSortBlock) s_h256[d] = 0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kNpl; ++i) {
                const uint32_t c = v[i];
                if (c != 0 && (c & pmask) == prefix) atomicAdd(&s_h256[(c >> shift) & 255u], 1u);
            }
            __syncthreads();
            if (wv == 0) {
                uint32_t h[4], hs = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h[q] = s_h256[255u - 4u * lane - q];
                    hs += h[q];
                }
                uint32_t tot;
                uint32_t above = wave_exscan_u32(hs, &tot);
                uint32_t sel = 0, nn = 0;
                bool found = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (!found && above < need && above + h[q] >= need) {
                        sel = 255u - 4u * lane - q;
                        nn = need - above;
                        found = true;
                    }
                    above += h[q];
                }
                const uint32_t fl = first_lane(ballot(found));
                if (lane == 0) {
                    s_t = rdlane(sel, fl);
                    s_take = rdlane(nn, fl);
                }
            }
            __syncthreads();
            prefix |= s_t << shift;
            pmask |= 0xFFu << shift;
            need = s_take;
        }
        __syncthreads();
        if (tid == 0) {
            s_t = prefix;
            s_take = need;
        }
        __syncthreads();
    }
    const uint32_t t = s_t, take_eq = s_take;

    // 2. ordered compaction from the registers (entry lo + 64 i + lane is in key order)
    {
        uint32_t gt = 0, eq = 0;  // per lane
#pragma unroll
        for (int i = 0; i < kNpl; ++i) {
            gt += v[i] > t;
            eq += v[i] == t;
        }
        gt = wave_sum_u32(gt);
        eq = wave_sum_u32(eq);
        if (lane == 0) {
            s_w[wv][0] = gt;
            s_w[wv][1] = eq;
        }
    }
    __syncthreads();
    {
        uint32_t eq_before = 0, sel_before = 0;
        for (uint32_t q = 0; q < wv; ++q) {
            const uint32_t eqq = s_w[q][1];
            const uint32_t left = take_eq > eq_before ? take_eq - eq_before : 0u;
            sel_before += s_w[q][0] + (eqq < left ? eqq : left);
            eq_before += eqq;
        }
        uint32_t running = sel_before, eq_seen = eq_before;
        const uint64_t lt = lanemask_lt();
#pragma unroll
        for (int i = 0; i < kNpl; ++i) {
            const uint32_t c = v[i];
            const uint64_t meq = ballot(c == t);
            const uint32_t eq_rank = (uint32_t)__popcll(meq & lt);
            const bool sel = c > t || (c == t && eq_seen + eq_rank < take_eq);
            const uint64_t ms = ballot(sel);
            const uint32_t pos = running + (uint32_t)__popcll(ms & lt);
            if (sel && pos < M) s_buf[0][pos] = make_uint2(c, lo + 64u * i + lane);
            running += (uint32_t)__popcll(ms);
            eq_seen += (uint32_t)__popcll(meq);
            __builtin_amdgcn_sched_barrier(0);  // one element's masks live at a time
        }
    }
    __syncthreads();

    // 3. stable LSD radix sort by v = mx - count in LDS
    const uint32_t range = mx - t;
    const uint32_t bits = range ? 32u - (uint32_t)__clz(range) : 0u;
    const uint32_t passes = (bits + 7u) / 8u;
    const uint32_t espan = (((M + kSortNW - 1) / kSortNW) + 63u) & ~63u;
    const uint32_t elo = wv * espan < M ? wv * espan : M, ehi = elo + espan < M ? elo + espan : M;
    uint32_t sb = 0;
    for (uint32_t pass = 0; pass < passes; ++pass) {
        const uint2* src = s_buf[sb];
        uint2* dst = s_buf[sb ^ 1u];
        const uint32_t shift = 8u * pass;
        for (uint32_t d = lane; d < 256; d += 64) s_hist[wv][d] = 0;
        for (uint32_t e = elo + lane; e < ehi; e += 64) atomicAdd(&s_hist[wv][((mx - src[e].x) >> shift) & 255u], 1u);
        __syncthreads();
        {  // offsets in (digit, wavefront) order: thread tid owns digit tid / 4, waves 4 (tid % 4) ..
            const uint32_t d = tid >> 2, x0 = (tid & 3u) * 4u;
            uint32_t hv[4], hs = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                hv[q] = s_hist[x0 + q][d];
                hs += hv[q];
            }
            __shared__ uint32_t s_scan[16];
            uint32_t tot;
            uint32_t ex = block_exscan_u32(hs, s_scan, &tot);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s_hist[x0 + q][d] = ex;
                ex += hv[q];
            }
        }
        __syncthreads();
        for (uint32_t e0 = elo; e0 < ehi; e0 += 64) {
            const uint32_t e = e0 + lane;
            const bool valid = e < ehi;
            const uint2 kv = valid ? src[e] : make_uint2(0u, 0u);
            const uint32_t d = valid ? ((mx - kv.x) >> shift) & 255u : 0u;
            uint64_t peers = ballot(valid);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool on = (d >> bit) & 1u;
                const uint64_t bb = ballot(on);
                peers &= on ? bb : ~bb;
            }
            const uint32_t rk = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t at = valid ? s_hist[wv][d] + rk : 0u;
            if (valid && at < M) dst[at] = kv;
            if (valid && rk == 0) atomicAdd(&s_hist[wv][d], (uint32_t)__popcll(peers));
        }
        __syncthreads();
        sb ^= 1u;
    }
    uint32_t* __restrict__ ord = order + (uint64_t)w * Cmax;
    uint32_t* __restrict__ ocnt = order_count + (uint64_t)w * Cmax;
    for (uint32_t e = tid; e < M; e += kSortBlock) {
        const uint2 kv = s_buf[sb][e];
        ord[e] = kv.y;
        ocnt[e] = kv.x;
    }
}

// ---------------------------------------------------------------------------------------
// Rows of kWideKeys keys and more, and kWideKeysPerWindow more for every window (C_max >= kWideCmax):
// the same order by many blocks per window. (One window of 66,000 keys: 65 us by one block, 69 by
// many; 90,000: 90 and 71; 200 windows of 66,000, which fill the chip by themselves: 101 and 177.)
// A row of a million counts kept one CU busy for 3.1 ms (its reads of 4 MB one after
// another, then three radix passes over 524,288 entries), while the other 255 idled.
//   k_wide_hist     histogram of the row over 1,728 bins that are exact below 128 and 1/64 of
//                   an octave wide above; row sum and maximum
//   k_wide_refine   three launches: where the bin of the C_max-th count is wider than one
//                   count, histograms of its next 10, 10 and 5 bits (else they exit)
//   k_wide_count    threshold t; per tile, the counts above it and equal to it
//   k_wide_compact  kept entries in key order, at places from the tiles' prefix
//   k_wide_sort     C_max <= 4,096: one block per window, radix passes in LDS
//   k_wide_digits / k_wide_offsets / k_wide_scatter  else, per 11 bits of (max - count): digit
//                   counts per tile of 4,096 entries, their prefix over the tiles, and the
//                   stable scatter (passes past the range exit)
// Scratch: the window's two buffers in the workspace (its rows of order and order_count are
// written where entries are kept and nowhere else). Every launch is a few microseconds of latency: cr_admit of 1,920
// from 128,824 keys 326 -> 74 us, of 524,288 from 1,000,000 3,290 -> 365 us, 24 windows of
// 128,824 244 -> 155 us.
// ---------------------------------------------------------------------------------------
constexpr uint32_t kWideCmax = 1024;   // smallest C_max whose buffers hold the scratch
// Smallest row. 100 windows of 50,000 keys took 99 us with a block each (they fill the chip by
// themselves) and 162 us this way.
// From 113 windows on a block each fills the chip whatever the rows (1e6 Zipf keys: 100 windows 1,225
// us by one block each and 1,140 by many, 150 windows 1,250 and 1,685).
constexpr uint32_t kWideKeys = 73728, kWideKeysPerWindow = 1536, kWideWindows = 112;
constexpr uint32_t kWideBins = 1728;
constexpr uint32_t kWideSub = 1024;    // bins of a refinement: 10 bits
constexpr uint32_t kWideThreads = 256;
constexpr uint32_t kWideSmall = 4096;  // largest C_max sorted by one block
constexpr uint32_t kWideTile = 4096;   // entries per tile of a radix pass
constexpr uint32_t kWideDigits = 2048; // 11 bits

// Per window, in its second buffer.
struct WideHead {
    uint32_t mx, t, take, M;  // largest count, threshold, entries equal to it that are kept, entries kept
    uint32_t low[32];         // the last refinement's bins
};

// Keys per block: at most 129 blocks per row, and about 512 in all (the blocks of a row meet
// in its bins' atomics: 24 rows of 128,824 keys 51 us with 63 blocks a row, 17 with 19).
inline uint32_t wide_tile(uint32_t K, uint32_t NW)
{
    const uint64_t share = (uint64_t)K * NW / 512u;
    const uint64_t t = share > K / 128u ? share : K / 128u;
    const uint64_t u = ((t > K ? K : t) + 1023u) & ~1023ull;
    return u < 2048u ? 2048u : (uint32_t)u;
}

__device__ __forceinline__ uint32_t wide_bin(uint32_t c)
{
    if (c < 64u) return c;
    const uint32_t e = 31u - (uint32_t)__builtin_clz(c);
    return 64u + (e - 6u) * 64u + ((c >> (e - 6u)) & 63u);
}

// A window's two buffers (2 C_max words each): the bins and the second refinement's from the
// first's start, then, from the second buffer's start or past those bins, the head, the tiles'
// counts and the first refinement's bins. Compaction may fill the first buffer with entries: it
// needs the head and the tiles only; the radix passes' counters then lie where the tiles were.
constexpr uint32_t kWideTiles = 132;  // tiles of a row (at most 129: wide_tile)
constexpr uint32_t kWideHeadWords = sizeof(WideHead) / 4u;
static_assert(kWideBins + kWideSub + kWideHeadWords + 2u * kWideTiles + kWideSub <= 4u * kWideCmax &&
                  (kWideBins + kWideSub) % 2u == 0 && kWideHeadWords % 2u == 0,
              "the smallest buffers hold the scratch, tiles and entries aligned");

struct WideWin {
    uint32_t* bins;           // [kWideBins]
    uint32_t *sub1, *sub2;    // [kWideSub] each
    WideHead* head;
    uint2* tiles;             // [kWideTiles] {above, equal}
    uint32_t *ord, *ocnt;     // the window's rows of order and order_count
    uint2* b0;
    uint32_t* counters;       // [tile][kWideDigits], then the totals
};

__device__ __forceinline__ WideWin wide_win(uint2* buf, uint32_t* order, uint32_t* order_count, uint32_t Cmax, uint32_t w)
{
    uint2* b0 = buf + (uint64_t)w * 2u * Cmax;
    uint32_t* words = reinterpret_cast<uint32_t*>(b0);
    uint32_t* head = words + (2u * Cmax > kWideBins + kWideSub ? 2u * Cmax : kWideBins + kWideSub);
    uint32_t* tiles = head + kWideHeadWords;
    return WideWin{words, tiles + 2u * kWideTiles, words + kWideBins, reinterpret_cast<WideHead*>(head),
                   reinterpret_cast<uint2*>(tiles), order + (uint64_t)w * Cmax, order_count + (uint64_t)w * Cmax, b0, tiles};
}

// From the top of `nbins` bins down: the bin in which the need-th entry lies, and how many of
// it are needed. One wavefront; uniform results.
__device__ __forceinline__ uint32_t wide_select(const uint32_t* __restrict__ bins, uint32_t nbins, uint32_t& need)
{
    const uint32_t lane = lane_id();
    const uint32_t per = (nbins + 63u) / 64u;
    uint32_t sum = 0;
    for (uint32_t q = 0; q < per; ++q) {
        const uint32_t d = lane * per + q;
        sum += d < nbins ? bins[nbins - 1u - d] : 0u;
    }
    const uint32_t incl = wave_incl_scan_u32(sum);
    const uint32_t own = first_lane(ballot(incl >= need));  // need <= the bins' total
    uint32_t above = rdlane(incl - sum, own);
    for (uint32_t q = 0;; ++q) {
        const uint32_t b = nbins - 1u - (own * per + q);
        const uint32_t h = bins[b];
        if (above + h >= need) {
            need -= above;
            return b;
        }
        above += h;
    }
}

// What the levels known so far say of the threshold: counts in [base, base + 2^bits) hold it,
// with `need` entries kept of them (bits = 0: the threshold is base). One wavefront.
struct WideSel {
    uint32_t base, bits, need, M;
};

__device__ __forceinline__ WideSel wide_threshold(const WideWin& ww, uint32_t Cmax, int levels)
{
    const uint32_t lane = lane_id();
    uint32_t nnz = 0;
    for (uint32_t b = 1u + lane; b < kWideBins; b += 64u) nnz += ww.bins[b];
    nnz = rdlane(wave_incl_scan_u32(nnz), 63u);
    if (nnz <= Cmax) return WideSel{0u, 0u, 0u, nnz};  // every nonzero key
    WideSel s{0u, 0u, Cmax, Cmax};
    const uint32_t b = wide_select(ww.bins, kWideBins, s.need);
    if (b < 128u) {
        s.base = b;
        return s;
    }
    s.bits = (b - 64u) / 64u;
    s.base = (64u | (b & 63u)) << s.bits;
    for (int l = 1; l < levels && s.bits; ++l) {
        const uint32_t rest = s.bits > 10u && l < 3 ? s.bits - 10u : 0u;
        const uint32_t d = wide_select(l == 1 ? ww.sub1 : (l == 2 ? ww.sub2 : ww.head->low), 1u << (s.bits - rest), s.need);
        s.base += d << rest;
        s.bits = rest;
    }
    return s;
}

__global__ __launch_bounds__(kWideThreads) void k_wide_zero(uint32_t Cmax, uint32_t* __restrict__ order,
                                                            uint32_t* __restrict__ order_count, uint2* __restrict__ buf,
                                                            uint64_t* __restrict__ row_sum)
{
    const uint32_t w = blockIdx.x;
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    for (uint32_t b = threadIdx.x; b < kWideBins; b += kWideThreads) ww.bins[b] = 0u;
    for (uint32_t b = threadIdx.x; b < kWideSub; b += kWideThreads) {
        ww.sub1[b] = 0u;
        ww.sub2[b] = 0u;
    }
    uint32_t* h = reinterpret_cast<uint32_t*>(ww.head);
    if (threadIdx.x < sizeof(WideHead) / 4u) h[threadIdx.x] = 0u;
    if (threadIdx.x == 0) row_sum[w] = 0ull;
}

__global__ __launch_bounds__(kWideThreads) void k_wide_hist(const uint32_t* __restrict__ counts, uint32_t K, uint32_t tile,
                                                            uint32_t Cmax, uint32_t* __restrict__ order,
                                                            uint32_t* __restrict__ order_count, uint2* __restrict__ buf,
                                                            uint64_t* __restrict__ row_sum)
{
    __shared__ uint32_t s_h[kWideBins];
    const uint32_t w = blockIdx.y, tid = threadIdx.x;
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    const uint32_t* __restrict__ row = counts + (uint64_t)w * K;
    const bool vec = (((uintptr_t)row) & 15u) == 0;
    for (uint32_t b = tid; b < kWideBins; b += kWideThreads) s_h[b] = 0u;
    __syncthreads();
    const uint32_t lo = blockIdx.x * tile, hi = K - lo < tile ? K : lo + tile;  // lo < K
    uint32_t mx = 0, n1 = 0, n2 = 0, n3 = 0;  // the bulk of a long tail without LDS atomics
    uint64_t sum = 0;
    for (uint32_t b = lo + 4u * tid; b < hi; b += 4u * kWideThreads) {
        const uint4 q = load4(row, hi, b, vec);
        const uint32_t cs[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t c = cs[u];
            n1 += c == 1u;
            n2 += c == 2u;
            n3 += c == 3u;
            mx = c > mx ? c : mx;
            sum += c;
            if (c >= 4u) atomicAdd(&s_h[wide_bin(c)], 1u);
        }
    }
    n1 = wave_sum_u32(n1);
    n2 = wave_sum_u32(n2);
    n3 = wave_sum_u32(n3);
    mx = wave_max_u32(mx);
    sum = wave_sum_u64(sum);
    if (lane_id() == 0) {
        if (n1) atomicAdd(&s_h[1], n1);
        if (n2) atomicAdd(&s_h[2], n2);
        if (n3) atomicAdd(&s_h[3], n3);
        if (mx) atomicMax(&ww.head->mx, mx);
        if (sum) atomicAdd(reinterpret_cast<unsigned long long*>(row_sum + w), (unsigned long long)sum);
    }
    __syncthreads();
    for (uint32_t b = 1u + tid; b < kWideBins; b += kWideThreads)
        if (s_h[b]) atomicAdd(&ww.bins[b], s_h[b]);
}

template <int kLevel>
__global__ __launch_bounds__(kWideThreads) void k_wide_refine(const uint32_t* __restrict__ counts, uint32_t K,
                                                              uint32_t tile, uint32_t Cmax, uint32_t* __restrict__ order,
                                                              uint32_t* __restrict__ order_count, uint2* __restrict__ buf)
{
    __shared__ uint32_t s_h[kWideSub];
    __shared__ WideSel s_sel;
    const uint32_t w = blockIdx.y, tid = threadIdx.x;
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    if (tid < 64u) {
        const WideSel s = wide_threshold(ww, Cmax, kLevel);
        if (tid == 0) s_sel = s;
    }
    for (uint32_t b = tid; b < kWideSub; b += kWideThreads) s_h[b] = 0u;
    __syncthreads();
    const WideSel s = s_sel;
    if (s.bits == 0u) return;
    const uint32_t rest = s.bits > 10u && kLevel < 3 ? s.bits - 10u : 0u;
    const uint32_t* __restrict__ row = counts + (uint64_t)w * K;
    const uint32_t lo = blockIdx.x * tile, hi = K - lo < tile ? K : lo + tile;
    for (uint32_t b = lo + tid; b < hi; b += kWideThreads) {
        const uint32_t u = row[b] - s.base;  // wraps below base
        if (u >> s.bits == 0u) atomicAdd(&s_h[u >> rest], 1u);
    }
    __syncthreads();
    uint32_t* __restrict__ out = kLevel == 1 ? ww.sub1 : (kLevel == 2 ? ww.sub2 : ww.head->low);
    for (uint32_t b = tid; b < 1u << (s.bits - rest); b += kWideThreads)
        if (s_h[b]) atomicAdd(&out[b], s_h[b]);
}

__global__ __launch_bounds__(kWideThreads) void k_wide_count(const uint32_t* __restrict__ counts, uint32_t K, uint32_t tile,
                                                             uint32_t Cmax, uint32_t* __restrict__ order,
                                                             uint32_t* __restrict__ order_count,
                                                             uint32_t* __restrict__ n_order, uint2* __restrict__ buf)
{
    __shared__ WideSel s_sel;
    __shared__ uint32_t s_gt, s_eq;
    const uint32_t w = blockIdx.y, tid = threadIdx.x;
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    if (tid < 64u) {
        const WideSel s = wide_threshold(ww, Cmax, 4);
        if (tid == 0) {
            s_sel = s;
            s_gt = 0;
            s_eq = 0;
        }
    }
    __syncthreads();
    const WideSel s = s_sel;
    const uint32_t* __restrict__ row = counts + (uint64_t)w * K;
    const bool vec = (((uintptr_t)row) & 15u) == 0;
    const uint32_t lo = blockIdx.x * tile, hi = K - lo < tile ? K : lo + tile;
    uint32_t gt = 0, eq = 0;
    for (uint32_t b = lo + 4u * tid; b < hi; b += 4u * kWideThreads) {
        const uint4 q = load4(row, hi, b, vec);
        gt += (q.x > s.base) + (q.y > s.base) + (q.z > s.base) + (q.w > s.base);
        eq += (q.x == s.base) + (q.y == s.base) + (q.z == s.base) + (q.w == s.base);  // past hi only for base 0: none kept
    }
    gt = wave_sum_u32(gt);
    eq = wave_sum_u32(eq);
    if (lane_id() == 0) {
        atomicAdd(&s_gt, gt);
        atomicAdd(&s_eq, eq);
    }
    __syncthreads();
    if (tid == 0) {
        ww.tiles[blockIdx.x] = make_uint2(s_gt, s_eq);
        if (blockIdx.x == 0) {
            ww.head->t = s.base;
            ww.head->take = s.need;
            ww.head->M = s.M;
            n_order[w] = s.M;
        }
    }
}

// 11-bit radix passes that the range of the kept counts takes.
__device__ __forceinline__ uint32_t wide_passes(const WideHead& h)
{
    const uint32_t range = h.M ? h.mx - (h.t ? h.t : 1u) : 0u;
    const uint32_t bits = range ? 32u - (uint32_t)__builtin_clz(range) : 0u;
    return (bits + 10u) / 11u;
}

// Kept entries in key order into the first buffer, or, for an even number of radix passes by
// many blocks, into order and order_count, where the last pass has to end.
__global__ __launch_bounds__(kWideThreads) void k_wide_compact(const uint32_t* __restrict__ counts, uint32_t K, uint32_t tile,
                                                               uint32_t Cmax, uint32_t* __restrict__ order,
                                                               uint32_t* __restrict__ order_count, uint2* __restrict__ buf)
{
    constexpr uint32_t kWaves = kWideThreads / 64u;
    __shared__ uint32_t s_w[kWaves][2];
    const uint32_t w = blockIdx.y, lane = lane_id(), wv = wave_in_block();
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    const uint32_t t = ww.head->t, take = ww.head->take, M = ww.head->M;
    if (M == 0) return;
    const bool soa = Cmax > kWideSmall && (wide_passes(*ww.head) & 1u) == 0u;
    uint32_t gt0 = 0, eq0 = 0;  // in the tiles before
    for (uint32_t q = lane; q < blockIdx.x; q += 64u) {
        const uint2 c = ww.tiles[q];
        gt0 += c.x;
        eq0 += c.y;
    }
    gt0 = wave_sum_u32(gt0);
    eq0 = wave_sum_u32(eq0);
    const uint32_t* __restrict__ row = counts + (uint64_t)w * K;
    const uint32_t lo = blockIdx.x * tile, hi = K - lo < tile ? K : lo + tile;
    const uint32_t span = tile / kWaves;  // a multiple of 64
    const uint32_t a = lo + wv * span < hi ? lo + wv * span : hi, z = a + span < hi ? a + span : hi;
    uint32_t gt = 0, eq = 0;
    for (uint32_t b = a + lane; b < z; b += 64u) {
        const uint32_t c = row[b];
        gt += c > t;
        eq += c == t;
    }
    gt = wave_sum_u32(gt);
    eq = wave_sum_u32(eq);
    if (lane == 0) {
        s_w[wv][0] = gt;
        s_w[wv][1] = eq;
    }
    __syncthreads();
    for (uint32_t q = 0; q < wv; ++q) {
        gt0 += s_w[q][0];
        eq0 += s_w[q][1];
    }
    uint32_t at = gt0 + (eq0 < take ? eq0 : take);
    for (uint32_t base = a; base < z; base += 64u) {
        const uint32_t b = base + lane;
        const uint32_t c = b < z ? row[b] : 0u;
        const uint64_t meq = ballot(b < z && c == t);
        const bool sel = b < z && (c > t || (c == t && eq0 + (uint32_t)__popcll(meq & lanemask_lt()) < take));
        const uint64_t ms = ballot(sel);
        const uint32_t pos = at + (uint32_t)__popcll(ms & lanemask_lt());
        if (sel && pos < M) {
            if (soa) {
                ww.ord[pos] = b;
                ww.ocnt[pos] = c;
            } else {
                ww.b0[pos] = make_uint2(c, b);
            }
        }
        at += (uint32_t)__popcll(ms);
        eq0 += (uint32_t)__popcll(meq);
    }
}

// C_max <= kWideSmall: stable LSD radix sort by (max - count) in LDS, as in k_sort_window_reg.
__global__ __launch_bounds__(kSortBlock) void k_wide_sort(uint32_t Cmax, uint32_t* __restrict__ order,
                                                          uint32_t* __restrict__ order_count, uint2* __restrict__ buf)
{
    extern __shared__ uint2 s_ent[];  // [2][Cmax]
    __shared__ uint32_t s_hist[kSortNW][256];
    __shared__ uint32_t s_scan[16];
    const uint32_t w = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wv = wave_in_block();
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    const uint32_t M = ww.head->M, mx = ww.head->mx, t = ww.head->t;
    if (M == 0) return;
    for (uint32_t e = tid; e < M; e += kSortBlock) s_ent[e] = ww.b0[e];
    __syncthreads();
    const uint32_t range = mx - t;
    const uint32_t bits = range ? 32u - (uint32_t)__builtin_clz(range) : 0u;
    const uint32_t passes = (bits + 7u) / 8u;
    const uint32_t espan = (((M + kSortNW - 1) / kSortNW) + 63u) & ~63u;
    const uint32_t elo = wv * espan < M ? wv * espan : M, ehi = elo + espan < M ? elo + espan : M;
    uint2* src = s_ent;
    uint2* dst = s_ent + Cmax;
    for (uint32_t pass = 0; pass < passes; ++pass) {
        const uint32_t shift = 8u * pass;
        for (uint32_t d = lane; d < 256; d += 64) s_hist[wv][d] = 0;
        for (uint32_t e = elo + lane; e < ehi; e += 64) atomicAdd(&s_hist[wv][((mx - src[e].x) >> shift) & 255u], 1u);
        __syncthreads();
        {  // offsets in (digit, wavefront) order: thread tid owns digit tid / 4, waves 4 (tid % 4) ..
            const uint32_t d = tid >> 2, x0 = (tid & 3u) * 4u;
            uint32_t hv[4], hs = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                hv[q] = s_hist[x0 + q][d];
                hs += hv[q];
            }
            uint32_t tot;
            uint32_t ex = block_exscan_u32(hs, s_scan, &tot);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s_hist[x0 + q][d] = ex;
                ex += hv[q];
            }
        }
        __syncthreads();
        for (uint32_t e0 = elo; e0 < ehi; e0 += 64) {
            const uint32_t e = e0 + lane;
            const bool valid = e < ehi;
            const uint2 kv = valid ? src[e] : make_uint2(0u, 0u);
            const uint32_t d = valid ? ((mx - kv.x) >> shift) & 255u : 0u;
            uint64_t peers = ballot(valid);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool on = (d >> bit) & 1u;
                const uint64_t bb = ballot(on);
                peers &= on ? bb : ~bb;
            }
            const uint32_t rk = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t at = valid ? s_hist[wv][d] + rk : 0u;
            if (valid && at < M) dst[at] = kv;
            if (valid && rk == 0) atomicAdd(&s_hist[wv][d], (uint32_t)__popcll(peers));
        }
        __syncthreads();
        uint2* tmp = src;
        src = dst;
        dst = tmp;
    }
    for (uint32_t e = tid; e < M; e += kSortBlock) {
        ww.ord[e] = src[e].y;
        ww.ocnt[e] = src[e].x;
    }
}

// One radix pass: entries of the pass's source, by index.
__device__ __forceinline__ uint2 wide_entry(const WideWin& ww, bool from_b0, uint32_t e)
{
    return from_b0 ? ww.b0[e] : make_uint2(ww.ocnt[e], ww.ord[e]);
}

__global__ __launch_bounds__(kWideThreads) void k_wide_digits(uint32_t Cmax, uint32_t pass, uint32_t* __restrict__ order,
                                                              uint32_t* __restrict__ order_count, uint2* __restrict__ buf)
{
    __shared__ uint32_t s_h[kWideDigits];
    const uint32_t w = blockIdx.y, tid = threadIdx.x;
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    const uint32_t M = ww.head->M, mx = ww.head->mx, np = wide_passes(*ww.head);
    const uint32_t e0 = blockIdx.x * kWideTile;
    if (pass >= np || e0 >= M) return;
    const bool from_b0 = ((np - pass) & 1u) != 0u;  // the last pass ends in order and order_count
    for (uint32_t d = tid; d < kWideDigits; d += kWideThreads) s_h[d] = 0u;
    __syncthreads();
    const uint32_t e1 = M - e0 < kWideTile ? M : e0 + kWideTile;
    for (uint32_t e = e0 + tid; e < e1; e += kWideThreads)
        atomicAdd(&s_h[((mx - (from_b0 ? ww.b0[e].x : ww.ocnt[e])) >> (11u * pass)) & (kWideDigits - 1u)], 1u);
    __syncthreads();
    uint32_t* __restrict__ out = ww.counters + (uint64_t)blockIdx.x * kWideDigits;
    for (uint32_t d = tid; d < kWideDigits; d += kWideThreads) out[d] = s_h[d];
}

// Per digit, the exclusive prefix of its tile counts in place; the total after the tiles.
__global__ __launch_bounds__(64) void k_wide_offsets(uint32_t Cmax, uint32_t pass, uint32_t* __restrict__ order,
                                                     uint32_t* __restrict__ order_count, uint2* __restrict__ buf)
{
    const uint32_t w = blockIdx.y, d = blockIdx.x * 64u + threadIdx.x;
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    if (pass >= wide_passes(*ww.head)) return;
    const uint32_t nt = (ww.head->M + kWideTile - 1u) / kWideTile;
    uint32_t* __restrict__ c = ww.counters + d;
    uint32_t run = 0;
    for (uint32_t q0 = 0; q0 < nt; q0 += 8u) {
        uint32_t v[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) v[q] = q0 + q < nt ? c[(uint64_t)(q0 + q) * kWideDigits] : 0u;
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
            if (q0 + q < nt) c[(uint64_t)(q0 + q) * kWideDigits] = run;
            run += v[q];
        }
    }
    c[(uint64_t)nt * kWideDigits] = run;
}

// Stable scatter of a tile: every wavefront ranks its 1,024 entries in order, 64 at a time. The
// lanes of one digit find each other in LDS (a tag byte per digit names a representative lane,
// whose 64-bit mask collects them), and a counter per wavefront and digit carries the rank on.
__global__ __launch_bounds__(kWideThreads) void k_wide_scatter(uint32_t Cmax, uint32_t pass, uint32_t* __restrict__ order,
                                                               uint32_t* __restrict__ order_count, uint2* __restrict__ buf)
{
    constexpr uint32_t kWaves = kWideThreads / 64u, kChunks = kWideTile / kWideThreads;
    __shared__ uint32_t s_cnt[kWaves][kWideDigits];
    __shared__ uint8_t s_tag[kWaves][kWideDigits];
    __shared__ unsigned long long s_peer[kWaves][64];
    __shared__ uint32_t s_scan[16];
    const uint32_t w = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wv = wave_in_block();
    const WideWin ww = wide_win(buf, order, order_count, Cmax, w);
    const uint32_t M = ww.head->M, mx = ww.head->mx, np = wide_passes(*ww.head);
    const uint32_t e0 = blockIdx.x * kWideTile;
    if (pass >= np || e0 >= M) return;
    const bool from_b0 = ((np - pass) & 1u) != 0u;
    for (uint32_t d = lane; d < kWideDigits; d += 64u) s_cnt[wv][d] = 0u;
    const uint32_t a = e0 + wv * (kWideTile / kWaves);
    uint2 kv[kChunks];
    uint32_t dr[kChunks];  // digit | rank among the wavefront's entries of it << 16
#pragma unroll
    for (uint32_t m = 0; m < kChunks; ++m) {
        const uint32_t e = a + 64u * m + lane;
        kv[m] = e < M ? wide_entry(ww, from_b0, e) : make_uint2(0u, 0u);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t m = 0; m < kChunks; ++m) {
        const bool valid = a + 64u * m + lane < M;
        const uint32_t d = valid ? ((mx - kv[m].x) >> (11u * pass)) & (kWideDigits - 1u) : 0u;
        s_peer[wv][lane] = 0ull;
        if (valid) s_tag[wv][d] = (uint8_t)lane;
        wave_lds_fence();
        const uint32_t rep = valid ? s_tag[wv][d] : lane;
        if (valid) atomicOr(&s_peer[wv][rep], 1ull << lane);
        wave_lds_fence();
        const uint64_t peers = valid ? (uint64_t)s_peer[wv][rep] : 0ull;
        const uint32_t rk = (uint32_t)__popcll(peers & lanemask_lt());
        uint32_t old = 0;
        if (valid && rk == 0) old = atomicAdd(&s_cnt[wv][d], (uint32_t)__popcll(peers));
        const uint32_t leader = valid ? (uint32_t)__builtin_ctzll(peers) : lane;
        old = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(leader << 2), (int)old);
        dr[m] = d | ((old + rk) << 16);
        wave_lds_fence();
    }
    __syncthreads();
    // first output position of every (digit, wavefront): digits before, tiles before, wavefronts before
    const uint32_t nt = (M + kWideTile - 1u) / kWideTile;
    const uint32_t* __restrict__ tot = ww.counters + (uint64_t)nt * kWideDigits;
    const uint32_t* __restrict__ off = ww.counters + (uint64_t)blockIdx.x * kWideDigits;
    constexpr uint32_t kPer = kWideDigits / kWideThreads;
    uint32_t tv[kPer], sum = 0;
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        tv[q] = tot[kPer * tid + q];
        sum += tv[q];
    }
    uint32_t all;
    uint32_t ex = block_exscan_u32(sum, s_scan, &all);
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        const uint32_t d = kPer * tid + q;
        uint32_t at = ex + off[d];
        for (uint32_t u = 0; u < kWaves; ++u) {
            const uint32_t c = s_cnt[u][d];
            s_cnt[u][d] = at;
            at += c;
        }
        ex += tv[q];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t m = 0; m < kChunks; ++m) {
        if (a + 64u * m + lane >= M) continue;
        const uint32_t at = s_cnt[wv][dr[m] & 0xFFFFu] + (dr[m] >> 16);
        if (at >= M) continue;
        if (from_b0) {
            ww.ord[at] = kv[m].y;
            ww.ocnt[at] = kv[m].x;
        } else {
            ww.b0[at] = kv[m];
        }
    }
}

// One block per plan: Eq. 1, the prefix admission and the plan's key index (bit b % 64 of word
// b / 64 set for every admitted key b, and per word the key rank of its first admitted key, an
// exclusive scan of the word popcounts; built in LDS when the words fit, else with global
// atomics).
//
// Counts fall along the order, so k does, and from the first key with k = 1 on (found by a
// 64-way search) neither Eq. 1 nor a prefix sum is left: the keys that still fit are a count,
// and their member offsets rise by one. Only the keys before it go through the block's
// prefix sum. What is left is one streaming pass over the admitted keys (their counts'
// sum, member offsets and index bits), bound by what one CU reads and writes: 524,288 admitted
// of 1,000,000 keys took 2,340 us when every 512 keys passed four block scans, 221 us now;
// 1,920 admitted of 20,000 keys x 947 plans 21.9 -> 13.5 us.
//
// Up to kAdmitSmall keys to go through (slots or keys, whichever are fewer) blocks of 8 wavefronts:
// four fit on a CU, so the plans of a step of many intervals run in one round (900 plans of
// 1,000 keys and 10,000 slots 55 us, 66 with 16). Above, 16 wavefronts.
constexpr uint32_t kAdmitSmall = 8192;
constexpr uint32_t kKxLdsWords = 18432;  // 144 KB of bits: up to 1,179,648 keys

template <int kThreads>
__device__ void build_key_index(const uint32_t* __restrict__ ord, uint32_t A, uint32_t KW, uint64_t* __restrict__ kx,
                                uint32_t* s_bits, bool in_lds, uint32_t* s_scan)
{
    // in_lds: the bits are set already
    const uint32_t tid = threadIdx.x;
    if (!in_lds) {
        for (uint32_t w = tid; w < KW; w += kThreads) kx[2u * w] = 0ull;
        __threadfence();
        __syncthreads();
        for (uint32_t a = tid; a < A; a += kThreads) {
            const uint32_t b = ord[a];
            atomicOr(reinterpret_cast<unsigned long long*>(&kx[2u * (b >> 6)]), 1ull << (b & 63u));
        }
        __threadfence();
    }
    __syncthreads();
    uint32_t carry = 0;
    for (uint32_t w0 = 0; w0 < KW; w0 += kThreads) {
        const uint32_t w = w0 + tid;
        uint64_t bits = 0;
        if (w < KW)
            bits = in_lds ? (uint64_t)s_bits[2u * w] | ((uint64_t)s_bits[2u * w + 1u] << 32)
                          : __hip_atomic_load(&kx[2u * w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t tot;
        const uint32_t ex = block_exscan_u32((uint32_t)__popcll(bits), s_scan, &tot);
        if (w < KW) {
            kx[2u * w] = bits;
            kx[2u * w + 1u] = carry + ex;
        }
        carry += tot;
    }
}

template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_admit_plan(
    uint32_t R, uint32_t Cmax, uint32_t NW, uint32_t KW,
    const cr_plan_spec* __restrict__ specs, const uint32_t* __restrict__ order,
    const uint32_t* __restrict__ order_count, const uint32_t* __restrict__ n_order,
    const uint64_t* __restrict__ row_sum, uint32_t* __restrict__ num_admitted, uint64_t* __restrict__ cold,
    uint32_t* __restrict__ clamped, uint32_t* __restrict__ member_off, uint64_t* __restrict__ key_index,
    uint32_t* __restrict__ err)
{
    extern __shared__ uint32_t s_bits[];  // [2 KW] when KW <= kKxLdsWords
    __shared__ uint32_t s_scan[16];
    __shared__ unsigned long long s_carried;
    __shared__ uint32_t s_clamped, s_used;
    const uint32_t p = blockIdx.x, tid = threadIdx.x, lane = lane_id();
    const cr_plan_spec spec = specs[p];
    uint32_t* __restrict__ moff = member_off + (uint64_t)p * (Cmax + 1u);
    uint64_t* __restrict__ kx = key_index + (uint64_t)p * 2u * KW;
    const bool in_lds = KW <= kKxLdsWords;
    if (in_lds)
        for (uint32_t w = tid; w < 2u * KW; w += kThreads) s_bits[w] = 0u;
    if (tid == 0) {
        s_carried = 0;
        s_clamped = 0;
    }
    __syncthreads();
    const bool eq1 = spec.variant == CR_PLAN_FULL || spec.variant == CR_PLAN_REPLICATED;
    bool ok = spec.window < NW && spec.W >= 1 && (uint64_t)R * spec.W <= Cmax && spec.variant <= CR_PLAN_FLAT;
    // the flat variant admits nothing: its whole window is cold
    const uint32_t M = ok && spec.variant != CR_PLAN_FLAT ? n_order[spec.window] : 0u;
    // N_w: given, or (CR_WINDOW_SUM) the row's sum with the target relative to the mean load,
    // q_cap = (q_num / q_den) N_w / R, i.e. Eq. 1 with q_num N_w and q_den R
    const uint64_t nw = ok ? row_sum[spec.window] : 0ull;
    const bool rel = spec.n_window == CR_WINDOW_SUM;
    if (ok && !rel && spec.n_window != nw) ok = false;
    uint64_t q_num = spec.q_num, q_den = spec.q_den;
    if (ok && rel) {
        if (nw && q_num > 0x7FFFFFFFFFFFFFFFull / nw) ok = false;
        q_num *= nw;
        q_den *= R;
    }
    const uint64_t n_window = nw;
    if (ok && eq1 && M > 0 && (q_num == 0 || q_den == 0 || q_den >= (1ull << 31))) ok = false;
    if (!ok) {
        if (tid == 0) {
            num_admitted[p] = 0;
            cold[p] = 0;
            clamped[p] = 0;
            moff[0] = 0;
            atomicOr(err, CR_ERR_SPEC);
        }
        build_key_index<kThreads>(order, 0u, KW, kx, s_bits, in_lds, s_scan);
        return;
    }
    const uint64_t C = (uint64_t)R * spec.W;
    const uint32_t* __restrict__ ord = order + (uint64_t)spec.window * Cmax;
    const uint32_t* __restrict__ ocnt = order_count + (uint64_t)spec.window * Cmax;
    // keys [0, a1) have k > 1 before the clamp to R (affinity: one copy per admitted key)
    uint32_t a1 = 0;
    if (eq1) {
        uint32_t hi = M;  // every wavefront searches for itself
        while (a1 < hi) {
            const uint32_t stride = (hi - a1 + 63u) / 64u;
            const uint32_t a = a1 + lane * stride;
            const uint32_t nb = (uint32_t)__popcll(ballot(a < hi && (uint64_t)ocnt[a < hi ? a : a1] * q_den > q_num));
            if (nb == 0) break;  // a1 itself has k = 1
            const uint32_t top = a1 + nb * stride;
            a1 += (nb - 1u) * stride + 1u;
            hi = top < hi ? top : hi;
        }
    }
    uint32_t used = 0, A = 0;  // <= C
    bool full = false;
    for (uint32_t base = 0; base < a1 && !full; base += kThreads) {
        const uint32_t a = base + tid;
        const bool valid = a < a1;
        uint32_t k = 0;
        bool cl = false;
        if (valid) {
            const uint64_t num = (uint64_t)ocnt[a] * q_den;
            const uint64_t kk = num / q_num + (num % q_num != 0);
            cl = kk > R;
            k = cl ? R : (uint32_t)kk;
        }
        uint32_t ktot;
        const uint32_t ex = block_exscan_u32(k, s_scan, &ktot);  // <= kThreads R
        const bool adm = valid && (uint64_t)used + ex + k <= C;
        if (adm) moff[a] = used + ex;
        const uint64_t clm = ballot(adm && cl);
        if (lane == 0 && clm) atomicAdd(&s_clamped, (uint32_t)__popcll(clm));
        const uint32_t nvalid = a1 - base < (uint32_t)kThreads ? a1 - base : (uint32_t)kThreads;
        if ((uint64_t)used + ktot <= C) {
            A += nvalid;
            used += ktot;
        } else {  // the first key that does not fit ends admission
            uint32_t nadm;
            const uint32_t before = block_exscan_flag(adm, s_scan, &nadm);
            if (tid == 0) s_used = used;
            __syncthreads();
            if (adm && before + 1u == nadm) s_used = used + ex + k;
            __syncthreads();
            A += nadm;
            used = s_used;
            full = true;
        }
    }
    if (!full) {
        const uint64_t room = C - used;
        const uint32_t n1 = (uint64_t)(M - a1) < room ? M - a1 : (uint32_t)room;
        for (uint32_t i = tid; i < n1; i += kThreads) moff[a1 + i] = used + i;
        A = a1 + n1;
        used += n1;
    }
    uint64_t sum = 0;
#pragma unroll 4
    for (uint32_t a = tid; a < A; a += kThreads) {
        sum += ocnt[a];
        if (in_lds) {
            const uint32_t b = ord[a];
            atomicOr(&s_bits[b >> 5], 1u << (b & 31u));
        }
    }
    sum = wave_sum_u64(sum);
    if (lane == 0 && sum) atomicAdd(&s_carried, (unsigned long long)sum);
    __syncthreads();
    if (tid == 0) {
        moff[A] = used;
        num_admitted[p] = A;
        const uint64_t carried = s_carried;
        cold[p] = n_window >= carried ? n_window - carried : 0ull;
        clamped[p] = s_clamped;
    }
    build_key_index<kThreads>(ord, A, KW, kx, s_bits, in_lds, s_scan);
}

__device__ __forceinline__ uint32_t dpp_shl1(uint32_t old, uint32_t v)  // lane i <- lane i+1
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, 0x130, 0xF, 0xF, false);
}

__device__ __forceinline__ uint32_t dpp_shr1(uint32_t old, uint32_t v)  // lane i <- lane i-1
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, 0x138, 0xF, 0xF, false);
}

__device__ __forceinline__ double dpp_shl1_f64(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp_shl1((uint32_t)u, (uint32_t)u), hi = dpp_shl1((uint32_t)(u >> 32), (uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double dpp_shr1_f64(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp_shr1((uint32_t)u, (uint32_t)u), hi = dpp_shr1((uint32_t)(u >> 32), (uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

struct LptBatch {
    uint32_t key, cnt, off, end;
};

__device__ __forceinline__ LptBatch lpt_load(const uint32_t* __restrict__ ord, const uint32_t* __restrict__ ocnt,
                                             const uint32_t* __restrict__ moff, uint32_t a, uint32_t A)
{
    LptBatch b{0u, 0u, 0u, 0u};
    if (a < A) {
        b.key = ord[a];
        b.cnt = ocnt[a];
        b.off = moff[a];
        b.end = moff[a + 1];
    }
    return b;
}

// Key index entry of key b ({bits, rank of the word's first admitted key}); the key's
// rank is entry.y + popcount of the bits below b.
__device__ __forceinline__ ulonglong2 kx_entry(const uint64_t* __restrict__ kx, uint32_t b, bool valid)
{
    return valid ? *reinterpret_cast<const ulonglong2*>(kx + 2u * (b >> 6)) : make_ulonglong2(0ull, 0ull);
}

__device__ __forceinline__ uint32_t kx_rank(ulonglong2 e, uint32_t b)
{
    return (uint32_t)e.y + (uint32_t)__popcll(e.x & ((1ull << (b & 63u)) - 1ull));
}

// R <= 64: lane i holds the i-th smallest (L, r), so the least-loaded destinations are
// lanes 0..k-1.
// Consecutive single-copy jobs are placed in batches. Job t+q would take lane q exactly as
// the sequential picks do as long as, for every q, lane q's load is below every charged
// load L_q' + x_q' of the earlier lanes q' < q (lane q is then the least (L, r) pair when
// job t+q is placed); an exclusive prefix minimum across the lanes gives the longest such
// batch M in one pass, ties ending it. The M charged lanes are merged back by rank: every
// lane's new position is the number of lanes with a smaller (L, r), counted either by
// pairwise exchanges over all lanes (many charged lanes) or by one ballot pass per charged
// lane (few), and one forward lane permutation applies it. A full round (M = R, equal x,
// order kept) needs no permutation.
// A batch of one is a single pick: three compares give the insertion rank and a one-lane
// DPP shift opens the slot; a job with k > 1 pops k lanes and re-inserts each.
// Admitted keys sit in two 64-key batches so a batch of jobs may straddle the boundary;
// the member picked for job a is kept in LDS slot a mod 128 until its batch is retired.
struct LptRaw {
    uint32_t key, cnt, off, end;
};

// Unconditional loads (the index is clamped into the plan's rows; entries past A are
// garbage and every use is masked by a < A): a load under an exec mask merges with a zero
// default, and that merge makes the wavefront wait for the load on the spot.
__device__ __forceinline__ LptRaw lpt_raw(const uint32_t* __restrict__ ord, const uint32_t* __restrict__ ocnt,
                                          const uint32_t* __restrict__ moff, uint32_t a, uint32_t Cmax)
{
    const uint32_t i = a < Cmax ? a : Cmax - 1u;
    return LptRaw{ord[i], ocnt[i], moff[i], moff[i + 1u]};
}

// The key index entry of key b as {bits lo, bits hi, rank of the word's first admitted key}
// (12 bytes: a 16-byte load would leave a dead register that the compiler may reuse, and
// the reuse has to wait for the load). Word indices past KW read word 0.
__device__ __forceinline__ uint3 kx_entry3(const uint64_t* __restrict__ kx, uint32_t b, uint32_t KW)
{
    const uint32_t w = (b >> 6) < KW ? (b >> 6) : 0u;
    return *reinterpret_cast<const uint3*>(kx + 2u * w);
}

__device__ __forceinline__ uint32_t kx_rank3(uint3 e, uint32_t b)
{
    const uint64_t bits = ((uint64_t)e.y << 32) | e.x;
    return e.z + (uint32_t)__popcll(bits & ((1ull << (b & 63u)) - 1ull));
}

__device__ __forceinline__ uint32_t ds_permute_u32(uint32_t dst_lane, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_ds_permute((int)(dst_lane << 2), (int)v);
}

__device__ __forceinline__ double ds_permute_f64(uint32_t dst_lane, double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = ds_permute_u32(dst_lane, (uint32_t)u), hi = ds_permute_u32(dst_lane, (uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ uint32_t ds_bpermute_u32(uint32_t src_lane, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src_lane << 2), (int)v);
}

__device__ __forceinline__ double ds_bpermute_f64(uint32_t src_lane, double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = ds_bpermute_u32(src_lane, (uint32_t)u), hi = ds_bpermute_u32(src_lane, (uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// (o, orv) < (a, r) as 0 or 1, without branches
__device__ __forceinline__ uint32_t lt_pair(double o, uint32_t orv, double a, uint32_t r)
{
    return (uint32_t)((o < a) | ((o == a) & (orv < r)));
}

// Lane i of a 16-lane row receives lane (i - kK) mod 16 of the same row (DPP row_ror:kK).
template <int kK>
__device__ __forceinline__ uint32_t row_ror_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x120 + kK, 0xF, 0xF, true);  // every source is in range
}

template <int kK>
__device__ __forceinline__ double row_ror_f64(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = row_ror_u32<kK>((uint32_t)u), hi = row_ror_u32<kK>((uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// How many of the row rotations kKs of (ov, orv) are smaller than this lane's (a, r). One
// rotation at a time (a scheduling barrier after each): unrolled together, their compare
// masks outgrow the scalar registers.
template <int... kKs>
__device__ __forceinline__ uint32_t count_rotations(double a, uint32_t r, double ov, uint32_t orv,
                                                    std::integer_sequence<int, kKs...>)
{
    uint32_t c = 0;
    ((c += lt_pair(row_ror_f64<kKs>(ov), row_ror_u32<kKs>(orv), a, r), __builtin_amdgcn_sched_barrier(0)), ...);
    return c;
}

// DPP move of a double; lanes whose source is outside the pattern (or whose row is masked
// off) receive `fill`.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_f64(double v, double fill)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v), f = (uint64_t)__double_as_longlong(fill);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)f, (int)(uint32_t)u, kCtrl, kRowMask, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(f >> 32), (int)(uint32_t)(u >> 32), kCtrl,
                                                              kRowMask, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// min over lanes 0 .. lane-1 (+inf on lane 0)
__device__ __forceinline__ double wave_exclusive_min_f64(double v)
{
    const double inf = INFINITY;
    double s = dpp_f64<0x138, 0xF>(v, inf);  // wave_shr:1
    s = fmin(s, dpp_f64<0x111, 0xF>(s, inf));  // row_shr:1
    s = fmin(s, dpp_f64<0x112, 0xF>(s, inf));  // row_shr:2
    s = fmin(s, dpp_f64<0x114, 0xF>(s, inf));  // row_shr:4
    s = fmin(s, dpp_f64<0x118, 0xF>(s, inf));  // row_shr:8
    s = fmin(s, dpp_f64<0x142, 0xA>(s, inf));  // row_bcast:15 into rows 1 and 3
    s = fmin(s, dpp_f64<0x143, 0xC>(s, inf));  // row_bcast:31 into rows 2 and 3
    return s;
}

__global__ __launch_bounds__(64) void k_lpt_small(uint32_t KW, uint32_t R, uint32_t Cmax, uint32_t NW,
                                                  const cr_plan_spec* __restrict__ specs,
                                                  const uint32_t* __restrict__ order,
                                                  const uint32_t* __restrict__ order_count,
                                                  const uint32_t* __restrict__ num_admitted,
                                                  const uint64_t* __restrict__ cold,
                                                  const uint32_t* __restrict__ member_off,
                                                  const uint64_t* __restrict__ key_index,
                                                  uint16_t* __restrict__ members, double* __restrict__ load,
                                                  uint32_t* __restrict__ route)
{
    issue_priority_high();
    // member picked for single-copy job a in slot a mod 128; slots 128.. take the stores of
    // lanes >= R so that the round loop needs no divergent branch
    __shared__ uint32_t s_mem[192];
    const uint32_t p = blockIdx.x, lane = lane_id();
    const cr_plan_spec spec = specs[p];
    if (hash_placed(spec.variant)) return;  // placed by cr_place_hash
    const uint32_t A = (uint32_t)__builtin_amdgcn_readfirstlane((int)num_admitted[p]);
    const uint32_t w = spec.window < NW ? spec.window : 0u;
    const uint32_t* __restrict__ ord = order + (uint64_t)w * Cmax;
    const uint32_t* __restrict__ ocnt = order_count + (uint64_t)w * Cmax;
    const uint32_t* __restrict__ moff = member_off + (uint64_t)p * (Cmax + 1u);
    uint16_t* __restrict__ mem = members + (uint64_t)p * Cmax;
    const uint64_t* __restrict__ kx = key_index + (uint64_t)p * 2u * KW;
    uint32_t* __restrict__ rw = route + (uint64_t)p * Cmax;
    double Lv = lane < R ? (double)cold[p] / (double)R : INFINITY;
    uint32_t rv = lane < R ? lane : 0xFFFFu;
    // Three 64-job batches in registers: the one being placed (cur), the next (nxt: a batch of
    // jobs may reach into it) and the one after (nx2), loaded a whole batch before it is first
    // read. The three register sets take these roles in turn (the step below is inlined three
    // times), so a retired batch's registers are reloaded in place with no copy. What the
    // placement loop reads of the batches (kc, xc, mc, mn, coff) is derived when the previous
    // batch retires, before that retire issues its loads: every wait is then for loads issued
    // a batch earlier, and the loop reads no register a load wrote (a loop that stores and
    // reads such registers gets a wait for every outstanding load at its entry).
    LptRaw s0 = lpt_raw(ord, ocnt, moff, lane, Cmax);
    LptRaw s1 = lpt_raw(ord, ocnt, moff, 64 + lane, Cmax);
    LptRaw s2 = lpt_raw(ord, ocnt, moff, 128 + lane, Cmax);
    uint3 kxc = kx_entry3(kx, s0.key, KW);                  // needed when the batch retires
    uint32_t kc = lane < A ? s0.end - s0.off : 0u;         // k of the current batch's keys (0 past A)
    double xc = kc == 1 ? (double)s0.cnt : (double)s0.cnt / (double)(kc ? kc : 1u);
    // lane q: the count of job base+q (mc) or base+64+q (mn) if it is a single-copy job, else
    // ~0; the current batch's member offsets xor k (coff)
    uint32_t mc = kc == 1 ? s0.cnt : 0xFFFFFFFFu;
    uint32_t mn = s1.end - s1.off == 1 ? s1.cnt : 0xFFFFFFFFu;
    uint32_t coff = s0.off ^ kc;
    const uint64_t rmask = R >= 64 ? ~0ull : ((1ull << R) - 1ull);
    const uint32_t P2 = R <= 1u ? 1u : 1u << (32 - __builtin_clz(R - 1u));  // power of two >= R
    uint32_t base = 0, t = 0;
    // Places jobs until the current batch retires (true: cur now holds the batch after nx2,
    // nxt is current) or every job is placed (false, after the final retire).
    auto step = [&](LptRaw& cur, const LptRaw& nxt, const LptRaw& nx2) __attribute__((always_inline)) -> bool {
        while (base + t < A) {
            // the loop state is uniform; saying so keeps it (and the masks built from it) scalar
            t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            if (t >= 64) {  // retire the current batch; its registers take the batch after nx2
                const uint32_t fm = s_mem[(base + lane) & 127u];
                const uint32_t rk = kx_rank3(kxc, cur.key);
                const bool one = kc == 1, live = base + lane < A;
                const uint32_t roff = coff ^ kc;
                kc = base + 64 + lane < A ? nxt.end - nxt.off : 0u;
                xc = (double)nxt.cnt;
                if (ballot(kc > 1)) xc = kc > 1 ? (double)nxt.cnt / (double)kc : xc;
                mc = kc == 1 ? nxt.cnt : 0xFFFFFFFFu;
                mn = nx2.end - nx2.off == 1 ? nx2.cnt : 0xFFFFFFFFu;
                coff = nxt.off ^ kc;
                kxc = kx_entry3(kx, nxt.key, KW);
                if (live) {
                    if (one) mem[roff] = (uint16_t)fm;
                    rw[rk] = one ? (CR_ROUTE_SINGLE | fm) : (base + lane);
                }
                base += 64;
                t -= 64;
                cur = lpt_raw(ord, ocnt, moff, base + 128 + lane, Cmax);
                return true;
            }
            const uint32_t k = rdlane(kc, t);
            if (k == 1) {
                // lane q looks at job t+q: its count if it is a single-copy job, else ~0
                const uint32_t src = (lane + t) & 63u;
                const uint32_t c1 = ds_bpermute_u32(src, mc), c2 = ds_bpermute_u32(src, mn);
                const uint32_t cq = lane + t < 64u ? c1 : c2;
                const bool jq = lane < R && cq != 0xFFFFFFFFu && base + t + lane < A;
                const double a = Lv + (double)cq;  // lane q's load once charged with job t+q
                const double pm = wave_exclusive_min_f64(jq ? a : INFINITY);
                const uint64_t okm = ballot(jq && (lane == 0 || Lv < pm));
                const uint32_t M = ~okm ? (uint32_t)__builtin_ctzll(~okm) : 64u;
                if (M >= 2) {
                    if (lane < M) s_mem[(base + t + lane) & 127u] = rv;
                    bool round = false;
                    const uint32_t c0 = rdlane(cq, 0);
                    if (M == R) {
                        const double an = dpp_shl1_f64(a);
                        const uint32_t rn = dpp_shl1(rv, rv);
                        round = ballot(lane < R && cq != c0) == 0 && ballot(lane + 1 < R && an == a && rn < rv) == 0;
                    }
                    if (round) {
                        Lv = lane < R ? a : Lv;
                        t += M;
                        // Further full rounds of the same run: the next R jobs have the same x, so
                        // the batch test reduces to every load being below min L + x, and the
                        // order test to the charged loads keeping their (L, r) order.
                        // (c0 is a single-copy job's count, never ~0)
                        const uint64_t same_c = ballot(mc == c0 && base + lane < A);
                        const uint64_t same_n = ballot(mn == c0 && base + 64 + lane < A);
                        const double x0 = (double)c0;
                        while (t < 64) {
                            // jobs t .. t+R-1 must all be single-copy jobs of count c0
                            const uint32_t e = t + R;  // one past the last job of the round (<= 128)
                            const uint64_t need_c = (e >= 64 ? ~0ull : ((1ull << e) - 1ull)) & ~((1ull << t) - 1ull);
                            const uint64_t need_n = e > 64 ? (e >= 128 ? ~0ull : ((1ull << (e - 64)) - 1ull)) : 0ull;
                            if ((same_c & need_c) != need_c || (same_n & need_n) != need_n) break;
                            const double an = Lv + x0;
                            const double v0 = rdlane_f64(an, 0);
                            const double ann = dpp_shl1_f64(an);
                            const uint32_t rn2 = dpp_shl1(rv, rv);
                            if (ballot(lane < R && !(Lv < v0)) != 0 || ballot(lane + 1 < R && ann == an && rn2 < rv) != 0)
                                break;
                            s_mem[lane < R ? ((base + t + lane) & 127u) : 128u + lane] = rv;
                            Lv = lane < R ? an : Lv;
                            t += R;
                            t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
                        }
                        continue;
                    } else {
                        const bool charged = lane < M;
                        const double av = charged ? a : Lv;
                        uint32_t np = 0;
                        if (4u * M > P2) {
                            // All pairs: lane i counts the lanes with a smaller (L, r). The 15
                            // other lanes of its 16-lane row come by DPP row rotations; each other
                            // row of the power-of-two block that holds the R destinations is
                            // brought over once (lane i ^ x) and rotated the same way. Lanes >= R
                            // hold +inf and count for no one.
                            using Rot = std::integer_sequence<int, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15>;
                            np = count_rotations(av, rv, av, rv, Rot{});
                            for (uint32_t x = 16; x < P2; x += 16) {
                                const double sw = ds_bpermute_f64(lane ^ x, av);
                                const uint32_t sr = ds_bpermute_u32(lane ^ x, rv);
                                np += lt_pair(sw, sr, av, rv) + count_rotations(av, rv, sw, sr, Rot{});
                            }
                            np = lane < R ? np : lane;
                        } else {
                            // Few charged lanes: one pass per charged lane q. The lanes preceding
                            // lane q form a lane mask; uncharged lanes after q count it.
                            uint32_t cnt = 0;
                            const uint64_t unch = rmask & ~((M >= 64 ? ~0ull : (1ull << M) - 1ull));
                            auto pass = [&](uint32_t q) {
                                const double aq = rdlane_f64(av, q);
                                const uint32_t rq = rdlane(rv, q);
                                const uint64_t bm = ballot(av < aq) | (ballot(av == aq) & ballot(rv < rq));
                                cnt += __builtin_amdgcn_inverse_ballot_w64(unch & ~bm) ? 1u : 0u;
                                return (uint32_t)__popcll(bm & rmask);
                            };
                            uint32_t q = 0;
                            for (; q + 1 < M; q += 2) {
                                const uint32_t r0 = pass(q), r1 = pass(q + 1);
                                cnt = wrlane(wrlane(cnt, r0, q), r1, q + 1);
                            }
                            if (q < M) {
                                const uint32_t rl = pass(q);  // before cnt is read: pass() adds to it
                                cnt = wrlane(cnt, rl, q);
                            }
                            np = charged ? cnt : (lane < R ? lane - M + cnt : lane);
                        }
                        Lv = ds_permute_f64(np, av);
                        rv = ds_permute_u32(np, rv);
                    }
                    t += M;
                    continue;
                }
                const double x = rdlane_f64(xc, t);
                const double v0 = rdlane_f64(Lv, 0) + x;
                const uint32_t r0 = rdlane(rv, 0);
                if (lane == 0) s_mem[(base + t) & 127u] = r0;
                // rank of (v0, r0) among lanes 1..: three compares, each straight to a lane mask
                const uint64_t m_lt = ballot(Lv < v0), m_eq = ballot(Lv == v0), m_r = ballot(rv < r0);
                const uint32_t pos = (uint32_t)__popcll((m_lt | (m_eq & m_r)) & ~1ull);
                const double sl = dpp_shl1_f64(Lv);
                const uint32_t sr = dpp_shl1(rv, rv);
                const bool lt = lane < pos, eq = lane == pos;
                Lv = lt ? sl : (eq ? v0 : Lv);
                rv = lt ? sr : (eq ? r0 : rv);
            } else {
                const double x = rdlane_f64(xc, t);
                const uint32_t off = rdlane(coff, t) ^ k;
                if (lane < k) mem[off + lane] = (uint16_t)rv;
                const double vnew = Lv + x;  // meaningful on lanes < k
                const uint32_t rnew = rv;
                const double sL = __shfl(Lv, (int)((lane + k) & 63u), 64);
                const uint32_t sR = __shfl(rv, (int)((lane + k) & 63u), 64);
                Lv = lane + k < 64u ? sL : INFINITY;
                rv = lane + k < 64u ? sR : 0xFFFFu;
                for (uint32_t u = 0; u < k; ++u) {
                    const double v = rdlane_f64(vnew, u);
                    const uint32_t r = rdlane(rnew, u);
                    const uint64_t m_lt = ballot(Lv < v), m_eq = ballot(Lv == v), m_r = ballot(rv < r);
                    const uint32_t pos = (uint32_t)__popcll(m_lt | (m_eq & m_r));
                    const double up = dpp_shr1_f64(Lv);
                    const uint32_t upr = dpp_shr1(rv, rv);
                    const bool gt = lane > pos, eq = lane == pos;
                    Lv = gt ? up : (eq ? v : Lv);
                    rv = gt ? upr : (eq ? r : rv);
                }
            }
            ++t;
        }
        // retire what is left (the current batch, and the next one if a batch of jobs reached it)
        {
            const uint32_t fm = s_mem[(base + lane) & 127u];
            if (base + lane < A) {
                if (kc == 1) mem[cur.off] = (uint16_t)fm;
                rw[kx_rank3(kxc, cur.key)] = kc == 1 ? (CR_ROUTE_SINGLE | fm) : (base + lane);
            }
        }
        if (t > 64) {
            const uint32_t fm = s_mem[(base + 64 + lane) & 127u];
            if (lane < t - 64 && base + 64 + lane < A) {
                const uint32_t kn = nxt.end - nxt.off;
                if (kn == 1) mem[nxt.off] = (uint16_t)fm;
                rw[kx_rank3(kx_entry3(kx, nxt.key, KW), nxt.key)] = kn == 1 ? (CR_ROUTE_SINGLE | fm) : (base + 64 + lane);
            }
        }
        return false;
    };
    while (step(s0, s1, s2) && step(s1, s2, s0) && step(s2, s0, s1)) {
    }
    if (lane < R) load[(uint64_t)p * R + rv] = Lv;
}

// 64 < R <= 1024: one block of N threads (N = the power of two >= R) per plan; thread i
// holds the i-th smallest (L, r) pair in registers, and the sorted state is mirrored in LDS.
// Jobs are placed in batches, with the rule k_lpt_small uses: consecutive single-copy jobs
// t, t+1, ... take sorted positions 0, 1, ... while position q's load is below every load
// charged to the positions before it in the batch (position q is then the least (L, r) pair
// when job t+q is placed), found by a block-wide exclusive prefix minimum; ties end the
// batch. A job with k > 1 is a batch of its own that charges positions 0..k-1, its members in
// that order. After a batch the charged positions are merged back into the sorted state. Jobs
// of one count keep the positions they charge in order, so the charged list is one sorted run
// per count: up to kLptRuns of them are merged with the uncharged positions by a merge path
// (each element's rank in every other run by binary search in LDS); more, or in blocks below
// kLptRunsFrom threads, by a bitonic sort of all N pairs.
//
// The tail of the order is long runs of one count x. Placing them is popping the smallest of
// the pairs {(L_i + j x, i), j >= 0} J times, and as long as no load leaves the power of two
// that the smallest load lies in, every such sum is exact (all are multiples of its last bit,
// the counts too while the loads are below 2^53; from there on no epochs are taken).
// With L_0 the smallest load, write L_i = L_0 + e_i x + f_i, 0 <= f_i < x: in epoch e the loads
// in [L_0 + e x, L_0 + (e + 1) x) are charged, once each, in the order of (f_i, i) among the
// destinations with e_i <= e. So one sort by (f, i) serves up to kLptEpochs epochs (each a
// batch of its own otherwise): the epochs' sizes are prefix lengths of the sorted state, a
// job's place in its epoch is a count of active destinations before it (ballots), and the
// new state is that sort order followed by the destinations still ahead.
// Which jobs start such a run is a bit per job beside the ring, made at its refills, so that
// a batch pays one scalar compare for it; and where a batch's counts change is looked up only when its
// charged pairs are out of order: a batch is bound by its barriers and by what 16 wavefronts
// read from one CU's LDS (every read more was about 1 %).
// One plan of 524,288 jobs over 1,024 destinations (611 batches, 403 of them of one count): 3,980 us
// by batches alone, 2,020 us; 24 plans over 257 destinations 436 -> 231 us. Without long runs
// (99,328 distinct counts, 1,024 destinations) 1,133 -> 936 us, by the sort's DPP steps.
// Route words are written afterwards by k_route_words, in parallel.
constexpr uint32_t kLptEpochs = 64;
// Rounds of R that a run must cover for it, in blocks up to 256 threads and above. An epoch run
// costs about 8 us there (sort, three rounds of loads) against 1.5 to 2.5 us for a batch: with
// 2, 4 and 6 rounds 188, 202 and 212 us (128 destinations, 16,384 jobs, mostly short runs),
// 965, 908 and 896 us (65 destinations, 33,280 jobs, all loads within one count); above, 2 is best.
constexpr uint32_t kLptRoundsSmall = 4, kLptRounds = 2;
constexpr uint32_t kLptRuns = 3;       // sorted runs merged at once (2 and 4 measured slower)
constexpr int kLptRunsFrom = 512;      // block size from which that beats the sort (small blocks: 98 against 86 us)

template <int N>
struct LptBlockLds {
    double v[2][N];        // sorted state (double-buffered for the merge)
    uint32_t r[2][N];
    double cv[N];          // the batch's charged pairs (positions 0..M-1)
    uint32_t cr[N];
    uint32_t jc[2 * N];    // job ring: counts, member offsets, k (0 past A)
    uint32_t jo[2 * N];
    uint16_t jk[2 * N];
    double wmin[N / 64];   // per-wavefront minimum of the charged loads
    double l0a[N / 64];    // per-wavefront lane 0: charged load, load, destination
    double l0v[N / 64];
    uint32_t l0r[N / 64];
    uint32_t wfail[N / 64];  // per-wavefront first position that fails the batch rule
    uint32_t wuns[N / 64];   // per-wavefront: 1 some charged pairs are out of order, 2 of one count
    unsigned long long run[2 * N / 64];  // ring: the jobs that start a run of one count long enough for epochs
    uint32_t en[kLptEpochs + 2];         // destinations active in an epoch
};

// Number of pairs among (v[lo .. lo+len)) smaller than (x, rx); the list is sorted, and its
// place and length are uniform, so that every lane takes the same steps.
__device__ __forceinline__ uint32_t lower_bound_pair(const double* __restrict__ v, const uint32_t* __restrict__ r,
                                                     uint32_t lo, uint32_t len, double x, uint32_t rx)
{
    uint32_t b = lo;
    for (uint32_t n = len; n > 0;) {
        const uint32_t h = (n + 1u) >> 1;
        b += lt_pair(v[b + h - 1u], r[b + h - 1u], x, rx) ? h : 0u;
        n -= h;
    }
    return b - lo;
}

// Bitonic sort of the block's N pairs, one per thread; tv and tr are scratch. A lane's partner in
// its wavefront comes by DPP for 1, 2 and 8 lanes' distance, else by ds_bpermute.
template <uint32_t J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, uint32_t at)
{
    if (J == 1u) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
    if (J == 2u) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    if (J == 8u) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);  // row_ror:8
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(at ^ (J << 2)), (int)v);
}

// `flip`: the lane keeps the larger pair of the two.
__device__ __forceinline__ void sort_keep(double& v, uint32_t& r, double pv, uint32_t pr, bool flip)
{
    const bool pless = lt_pair(pv, pr, v, r) != 0;
    if (pless != flip) {
        v = pv;
        r = pr;
    }
}

template <uint32_t J>
__device__ __forceinline__ void wave_sort_step(double& v, uint32_t& r, uint32_t dir, uint32_t at)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = lane_xor<J>((uint32_t)b, at), hi = lane_xor<J>((uint32_t)(b >> 32), at);
    sort_keep(v, r, __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32))), lane_xor<J>(r, at), (dir & J) != 0u);
}

template <int N>
__device__ __forceinline__ void block_sort_round(double& v, uint32_t& r, double* tv, uint32_t* tr, uint32_t kk)
{
    const uint32_t i = threadIdx.x, at = (i & 63u) << 2;
    uint32_t dir = (i & kk) ? ~i : i;  // bit j: the step of distance j keeps the larger pair here
    asm volatile("" : "+v"(dir));      // (the steps' lane masks are made where they are used: all at once, they spill)
#pragma unroll 1
    for (uint32_t j = kk >> 1; j >= 64u; j >>= 1) {
        tv[i] = v;
        tr[i] = r;
        __syncthreads();
        const double pv = tv[i ^ j];
        const uint32_t pr = tr[i ^ j];
        __syncthreads();
        sort_keep(v, r, pv, pr, (dir & j) != 0u);
    }
    if (kk > 32u) wave_sort_step<32>(v, r, dir, at);
    if (kk > 16u) wave_sort_step<16>(v, r, dir, at);
    if (kk > 8u) wave_sort_step<8>(v, r, dir, at);
    if (kk > 4u) wave_sort_step<4>(v, r, dir, at);
    if (kk > 2u) wave_sort_step<2>(v, r, dir, at);
    wave_sort_step<1>(v, r, dir, at);
}

template <int N>
__device__ __forceinline__ void block_sort_pairs(double& v, uint32_t& r, double* tv, uint32_t* tr)
{
    if (N <= 256) {
#pragma unroll
        for (uint32_t kk = 2; kk <= N; kk <<= 1) block_sort_round<N>(v, r, tv, tr, kk);
    } else {
#pragma unroll 1
        for (uint32_t kk = 2; kk <= N; kk <<= 1) block_sort_round<N>(v, r, tv, tr, kk);
    }
}

template <int N>
__global__ __launch_bounds__(N) void k_lpt_block(uint32_t R, uint32_t Cmax, const cr_plan_spec* __restrict__ specs,
                                                 const uint32_t* __restrict__ order_count,
                                                 const uint32_t* __restrict__ num_admitted,
                                                 const uint64_t* __restrict__ cold, uint32_t NW,
                                                 const uint32_t* __restrict__ member_off,
                                                 uint16_t* __restrict__ members, double* __restrict__ load)
{
    static_assert(N >= 128 && N <= 1024 && (N & (N - 1)) == 0, "block of 128..1024 threads");
    constexpr uint32_t NWV = N / 64;
    __shared__ LptBlockLds<N> sh;
    issue_priority_high();
    const uint32_t p = blockIdx.x, i = threadIdx.x, lane = lane_id(), wv = i >> 6;
    const cr_plan_spec spec = specs[p];
    if (hash_placed(spec.variant)) return;  // placed by cr_place_hash
    const uint32_t A = num_admitted[p];
    const uint32_t w = spec.window < NW ? spec.window : 0u;
    const uint32_t* __restrict__ ocnt = order_count + (uint64_t)w * Cmax;
    const uint32_t* __restrict__ moff = member_off + (uint64_t)p * (Cmax + 1u);
    uint16_t* __restrict__ mem = members + (uint64_t)p * Cmax;
    const double INF = INFINITY;
    double v = i < R ? (double)cold[p] / (double)R : INF;
    uint32_t r = i < R ? i : 0xFFFFFFFFu;
    sh.v[0][i] = v;
    sh.r[0][i] = r;
    const uint32_t run_len = (N <= 256 ? kLptRoundsSmall : kLptRounds) * R;  // shortest run placed by epochs
    struct Job {
        uint32_t c, o, k, z;  // count, member offset, k (0 past A), count at the end of a run
    };
    auto job = [&](uint32_t a) {
        const uint32_t aa = a < A ? a : 0u;
        Job q;
        q.c = ocnt[aa];
        q.o = moff[aa];
        q.k = a < A ? moff[aa + 1] - q.o : 0u;
        q.z = ocnt[a + run_len <= A ? a + run_len - 1u : aa];
        return q;
    };
    auto put = [&](uint32_t a, const Job& q) {
        const uint32_t slot = a & (2u * N - 1u);
        sh.jc[slot] = q.c, sh.jo[slot] = q.o, sh.jk[slot] = (uint16_t)q.k;
        const uint64_t starts = ballot(q.k == 1u && a + run_len <= A && q.z == q.c);
        if (lane == 0) sh.run[slot >> 6] = starts;
    };
    const Job q0 = job(i), q1 = job(N + i);
    Job pre = job(2 * N + i);  // job base + 2N + i, loaded one refill ahead
    put(i, q0);
    put(N + i, q1);
    static_assert(kLptEpochs == 64 && kLptEpochs * NWV * 4u <= sizeof(sh.cv), "epochs by lane; counts in cv");
    uint32_t cur = 0, base = 0, t = 0;
    uint32_t next_run = 0;  // no job in t .. next_run - 1 starts a run to be placed by epochs
    __syncthreads();
    while (t < A) {
        const uint32_t rj = (t + i) & (2u * N - 1u), r0 = t & (2u * N - 1u);
        const uint32_t c = sh.jc[rj], o = sh.jo[rj], k = sh.jk[rj];
        const uint32_t k0 = sh.jk[r0];
        if (t >= next_run) {
            // the next job in the ring that starts such a run
            const uint32_t w0 = (t >> 6) + lane;
            uint64_t starts = w0 < (base >> 6) + 2u * NWV ? sh.run[w0 & (2u * NWV - 1u)] : 0ull;
            if (lane == 0) starts &= ~0ull << (t & 63u);
            const uint64_t any = ballot(starts != 0ull);
            const uint32_t u = any ? first_lane(any) : 0u;
            next_run = any ? ((t >> 6) + u) * 64u + (uint32_t)__builtin_ctzll(rdlane64(starts, u)) : base + 2u * N;
            if (t == next_run) {
                const uint32_t c0 = sh.jc[r0], o0 = sh.jo[r0];
                const double x = (double)c0, v0 = sh.v[cur][0];
                // epochs before a load may leave the power of two of v0
                const double top = __longlong_as_double((long long)(((((uint64_t)__double_as_longlong(v0)) >> 52) + 1ull) << 52));
                const double fit = (top - v0) / x - 2.0;
                const uint32_t emax = v0 >= 9007199254740992.0 ? 0u : (fit >= (double)kLptEpochs ? kLptEpochs : (fit >= 2.0 ? (uint32_t)fit : 0u));
                if (emax >= 2u) {
                    const uint64_t last = (uint64_t)t + (uint64_t)(lane + 1u) * R - 1u;
                    const uint32_t m = (uint32_t)__popcll(ballot(last < A && ocnt[last < A ? (uint32_t)last : t] == c0));
                    // the run's jobs, up to 64 R of them: m R, and those of the next R
                    const uint64_t more = (uint64_t)t + (uint64_t)m * R + i;
                    const uint64_t same = ballot(m < 64u && i < R && more < A && ocnt[more < A ? (uint32_t)more : t] == c0);
                    uint32_t e = emax + 1u;
                    double f = 0.0;
                    if (i < R && v < v0 + (double)(emax + 1u) * x) {
                        const double d = v - v0;
                        double q = floor(d / x);
                        f = d - q * x;
                        if (f < 0.0) q -= 1.0, f += x;
                        else if (f >= x) q += 1.0, f -= x;
                        e = (uint32_t)q;
                    }
                    sh.cr[i] = e;  // nondecreasing in i
                    if (lane == 0) sh.wfail[wv] = (uint32_t)__popcll(same);
                    __syncthreads();
                    const uint32_t en = i + 1u < (uint32_t)N ? sh.cr[i + 1u] : emax + 1u;
                    for (uint32_t u = e; u < en && u <= emax; ++u) sh.en[u] = i + 1u;
                    const uint32_t J = m * R + rdlane(wave_incl_scan_u32(lane < NWV ? sh.wfail[lane] : 0u), 63u);
                    __syncthreads();
                    // lane u: destinations active in epoch u and jobs before it; the epochs J covers
                    // whole (E of them, at least one) and what it takes of the next
                    const uint32_t na = lane < emax ? sh.en[lane] : 0u;
                    const uint32_t incl = wave_incl_scan_u32(na);
                    const uint32_t first = incl - na;
                    const uint32_t E = (uint32_t)__popcll(ballot(lane + 1u < emax && incl <= J));
                    const uint32_t whole = rdlane(incl, E - 1u), nE = sh.en[E];
                    const uint32_t left = J - whole < nE ? J - whole : 0u;
                    const uint32_t nP = sh.en[E + 1u];
                    double sf = i < nP ? f : INF;
                    uint32_t sr = i < nP ? (r << 7) | e : 0xFFFFFFFFu;
                    // the ring starts again around the next job: its loads run under the sort
                    t += whole + left;
                    base = t & ~(uint32_t)(N - 1);
                    const Job q0 = job(base + i), q1 = job(base + N + i);
                    pre = job(base + 2 * N + i);
                    block_sort_pairs<N>(sf, sr, sh.v[cur ^ 1u], sh.r[cur ^ 1u]);
                    const uint32_t se = sr & 127u;
                    const bool in = i < nP;
                    uint32_t* __restrict__ wc = reinterpret_cast<uint32_t*>(sh.cv);  // [epoch][wavefront]
                    uint32_t mine = 0;
                    for (uint32_t u = 0; u <= E; ++u) {
                        const uint32_t n = (uint32_t)__popcll(ballot(in && se <= u));
                        mine = lane == u ? n : mine;
                    }
                    wc[lane * NWV + wv] = mine;
                    __syncthreads();
                    uint32_t at = 0;  // lane u: epoch u's active destinations in earlier wavefronts
                    for (uint32_t u = 0; u < wv; ++u) at += wc[lane * NWV + u];
                    uint32_t place = 0;
                    for (uint32_t u = 0; u <= E; ++u) {
                        const bool on = in && se <= u;
                        const uint64_t om = ballot(on);
                        place = rdlane(at, u) + __builtin_amdgcn_mbcnt_hi((uint32_t)(om >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)om, 0u));
                        if (on && (u < E || place < left)) mem[o0 + rdlane(first, u) + place] = (uint16_t)(sr >> 7);
                    }
                    if (in) {
                        // epoch E's uncharged ones, then epoch E + 1's
                        const bool stay = se <= E && place >= left;
                        const uint32_t pos = stay ? place - left : nE - left + i - (place > left ? place - left : 0u);
                        sh.v[cur][pos] = (v0 + (double)(stay ? E : E + 1u) * x) + sf;
                        sh.r[cur][pos] = sr >> 7;
                    }
                    put(base + i, q0);
                    put(base + N + i, q1);
                    __syncthreads();
                    v = sh.v[cur][i];
                    r = sh.r[cur][i];
                    next_run = t;
                    continue;
                }
                next_run = t + R;
            }
        }
        double a;
        uint32_t M;
        if (k0 > 1) {
            // multi-copy job t: positions 0..k0-1, each charged count / k0
            const double x0 = (double)sh.jc[r0] / (double)k0;
            a = v + x0;
            if (lane == 0) {
                sh.l0a[wv] = a;
                sh.l0v[wv] = v;
                sh.l0r[wv] = r;
            }
            M = k0;
            if (i < M) mem[sh.jo[r0] + i] = (uint16_t)r;
            __syncthreads();
        } else {
            const bool single = k == 1 && i < R;
            a = single ? v + (double)c : INF;  // position i's load once charged with job t+i
            double pm = wave_exclusive_min_f64(a);
            const double wtot = rdlane_f64(fmin(pm, a), 63u);
            if (lane == 0) {
                sh.wmin[wv] = wtot;
                sh.l0a[wv] = a;
                sh.l0v[wv] = v;
                sh.l0r[wv] = r;
            }
            __syncthreads();
            for (uint32_t u = 0; u < wv; ++u) pm = fmin(pm, sh.wmin[u]);
            const bool ok = single && (i == 0 || v < pm);
            const uint64_t bad = ballot(!ok);
            if (lane == 0) sh.wfail[wv] = bad ? wv * 64u + (uint32_t)__builtin_ctzll(bad) : N;
            __syncthreads();
            M = N;
            for (uint32_t u = 0; u < NWV; ++u) M = min(M, sh.wfail[u]);
            if (i < M) mem[o] = (uint16_t)r;
        }
        M = (uint32_t)__builtin_amdgcn_readfirstlane((int)M);
        // charged pairs (positions < M) and whether they are still in (L, r) order
        const bool charged = i < M;
        const double wv_ = charged ? a : v;
        double nx = __shfl_down(wv_, 1, 64);
        uint32_t nr = __shfl_down(r, 1, 64);
        if (lane == 63 && wv + 1 < NWV) {
            nx = (wv + 1) * 64u < M ? sh.l0a[wv + 1] : sh.l0v[wv + 1];
            nr = sh.l0r[wv + 1];
        }
        const bool out_of_order = i + 1 < M && !lt_pair(wv_, r, nx, nr);
        const uint64_t uns = ballot(out_of_order);
        uint32_t flags = uns != 0 ? 1u : 0u;
        if (N >= kLptRunsFrom && uns) flags |= ballot(out_of_order && c == sh.jc[(t + i + 1u) & (2u * N - 1u)]) ? 2u : 0u;
        if (lane == 0) sh.wuns[wv] = flags;
        if (charged) {
            sh.cv[i] = a;
            sh.cr[i] = r;
        }
        __syncthreads();
        uint32_t any_uns = 0;
        for (uint32_t u = 0; u < NWV; ++u) any_uns |= sh.wuns[u];
        any_uns = (uint32_t)__builtin_amdgcn_readfirstlane((int)any_uns);
        const uint32_t nxt = cur ^ 1u;
        uint32_t nruns = any_uns ? kLptRuns + 1u : 1u;  // sorted runs of the charged list
        uint32_t rs[kLptRuns + 1];                      // and their starts
        if (N >= kLptRunsFrom && any_uns == 1u && k0 == 1) {
            // a run ends where the count changes: in at most two of 64 pieces of the batch, else
            // there are too many
            const uint32_t s = (M + 63u) / 64u, at = lane * s, to = at + s < M ? at + s : M - 1u;
            const uint64_t has = ballot(at + 1u < M && sh.jc[(t + at) & (2u * N - 1u)] != sh.jc[(t + to) & (2u * N - 1u)]);
            if (__popcll(has) < kLptRuns) {
                static_assert(kLptRuns == 3 && N <= 1024, "two pieces of up to 16 jobs by lane");
                const uint32_t piece = lane < 16u ? first_lane(has) : first_lane(has & (has - 1ull));
                const uint32_t e = piece * s + (lane & 15u);
                const bool in = lane < 16u * (uint32_t)__popcll(has) && (lane & 15u) < s && e + 1u < M;
                const uint64_t ends = ballot(in && sh.jc[(t + e) & (2u * N - 1u)] != sh.jc[(t + e + 1u) & (2u * N - 1u)]);
                nruns = 1u + (uint32_t)__popcll(ends);
                rs[1] = ends ? rdlane(e, first_lane(ends)) + 1u : M;
                rs[2] = ends & (ends - 1ull) ? rdlane(e, first_lane(ends & (ends - 1ull))) + 1u : M;
            }
        }
        if (nruns <= kLptRuns) {
            // merge path: the charged list cv[0..M), one sorted run or one per count, and the
            // unchanged sorted positions M..R-1
            if (i < R) {
                const double y = charged ? a : v;
                uint32_t pos = charged ? lower_bound_pair(sh.v[cur], sh.r[cur], M, R - M, y, r) : i - M;
                if (nruns == 1u) {
                    pos += charged ? i : lower_bound_pair(sh.cv, sh.cr, 0, M, y, r);
                } else {
                    rs[0] = 0;
                    rs[kLptRuns] = M;
#pragma unroll
                    for (uint32_t q = 0; q < kLptRuns; ++q) {
                        if (rs[q] >= rs[q + 1]) continue;
                        const bool own = charged && i >= rs[q] && i < rs[q + 1];
                        pos += own ? i - rs[q] : lower_bound_pair(sh.cv, sh.cr, rs[q], rs[q + 1] - rs[q], y, r);
                    }
                }
                sh.v[nxt][pos] = y;
                sh.r[nxt][pos] = r;
            } else {
                sh.v[nxt][i] = INF;
                sh.r[nxt][i] = 0xFFFFFFFFu;
            }
            __syncthreads();
            v = sh.v[nxt][i];
            r = sh.r[nxt][i];
        } else {
            // bitonic sort of all N pairs (positions >= R hold (+inf, ~0) and stay last)
            v = wv_;
            block_sort_pairs<N>(v, r, sh.v[nxt], sh.r[nxt]);
            sh.v[nxt][i] = v;
            sh.r[nxt][i] = r;
        }
        cur = nxt;
        t += k0 > 1 ? 1u : (M ? M : 1u);  // M = 0 only for a job with k = 0, which admission never makes
        if (t >= base + N) {  // the ring's older half is consumed: refill it one half ahead
            put(base + 2 * N + i, pre);
            base += N;
            pre = job(base + 2 * N + i);
        }
        __syncthreads();
    }
    if (i < R) load[(uint64_t)p * R + r] = v;
}

// Route words of plans placed by k_lpt_block: per admitted key a, CR_ROUTE_SINGLE | its
// member when k = 1, else a, stored at the key's rank in the plan's key index.
constexpr uint32_t kWordThreads = 256;

__global__ __launch_bounds__(kWordThreads) void k_route_words(uint32_t Cmax, uint32_t NW, uint32_t KW,
                                                              const cr_plan_spec* __restrict__ specs,
                                                              const uint32_t* __restrict__ order,
                                                              const uint32_t* __restrict__ num_admitted,
                                                              const uint32_t* __restrict__ member_off,
                                                              const uint16_t* __restrict__ members,
                                                              const uint64_t* __restrict__ key_index,
                                                              uint32_t* __restrict__ route)
{
    const uint32_t p = blockIdx.y;
    const uint32_t a = blockIdx.x * kWordThreads + threadIdx.x;
    const cr_plan_spec spec = specs[p];
    if (hash_placed(spec.variant) || a >= num_admitted[p]) return;
    const uint32_t w = spec.window < NW ? spec.window : 0u;
    const uint32_t b = order[(uint64_t)w * Cmax + a];
    const uint32_t* __restrict__ moff = member_off + (uint64_t)p * (Cmax + 1u);
    const uint32_t o = moff[a], k = moff[a + 1] - o;
    const uint32_t word = k == 1 ? (CR_ROUTE_SINGLE | members[(uint64_t)p * Cmax + o]) : a;
    const ulonglong2 e = kx_entry(key_index + (uint64_t)p * 2u * KW, b, (b >> 6) < KW);
    route[(uint64_t)p * Cmax + kx_rank(e, b)] = word;
}

// Hash placement of the ablation variants (Section 5.2, 8B component ablation table).
// Members do not depend on the loads, so they are found for every admitted key at once
// (k_hash_members, one thread per key: k passes over the R hashes, each taking the
// smallest u above the previous pick, since one key's u values are distinct); only the
// load sums are ordered, and one wavefront per plan adds them in admission order with
// the destinations spread over its lanes (k_hash_loads).
constexpr uint32_t kHashThreads = 256;
constexpr uint32_t kHashStage = 4096;  // largest Cmax whose lists k_hash_loads keeps in LDS

inline size_t hash_loads_lds_bytes(uint32_t Cmax) { return (size_t)Cmax * 14u + 2u + 512u; }

__device__ __forceinline__ uint32_t place_key_hash(uint32_t seed, uint32_t b)
{
    return fmix32(b ^ fmix32(seed ^ 0x7F4A7C15u));
}

__global__ void __launch_bounds__(kHashThreads)
    k_hash_members(uint32_t R, uint32_t Cmax, uint32_t NW, uint32_t KW, const cr_plan_spec* __restrict__ specs,
                   const uint32_t* __restrict__ order, const uint32_t* __restrict__ num_admitted,
                   const uint32_t* __restrict__ member_off, const uint64_t* __restrict__ key_index,
                   uint16_t* __restrict__ members, uint32_t* __restrict__ route)
{
    const uint32_t p = blockIdx.x;
    const uint32_t variant = specs[p].variant;
    if (!hash_placed(variant)) return;
    const uint32_t A = min(num_admitted[p], Cmax);
    const uint32_t a = blockIdx.y * kHashThreads + threadIdx.x;
    if (a >= A) return;
    const uint32_t w = min(specs[p].window, NW - 1u);  // A > 0 only for a valid window
    const uint32_t b = order[(uint64_t)w * Cmax + a];
    const uint32_t* __restrict__ moff = member_off + (uint64_t)p * (Cmax + 1u);
    const uint32_t o = moff[a], k = moff[a + 1u] - o;
    const uint32_t kb = place_key_hash(specs[p].place_seed, b);
    uint16_t* __restrict__ mem = members + (uint64_t)p * Cmax + o;
    uint32_t prev = 0, first = 0;
    for (uint32_t t = 0; t < k; ++t) {
        uint32_t best_u = 0, best_r = R;
        for (uint32_t r = 0; r < R; ++r) {
            const uint32_t u = fmix32(kb ^ r);
            if ((t == 0 || u > prev) && (best_r == R || u < best_u)) {
                best_u = u;
                best_r = r;
            }
        }
        mem[t] = (uint16_t)best_r;
        prev = best_u;
        if (t == 0) first = best_r;
    }
    const ulonglong2 e = kx_entry(key_index + (uint64_t)p * 2u * KW, b, true);
    route[(uint64_t)p * Cmax + kx_rank(e, b)] = k == 1u ? (CR_ROUTE_SINGLE | first) : a;
}

template <int kS>
__global__ void __launch_bounds__(64)
    k_hash_loads(uint32_t R, uint32_t Cmax, uint32_t NW, const cr_plan_spec* __restrict__ specs,
                 const uint32_t* __restrict__ order_count, const uint32_t* __restrict__ num_admitted,
                 const uint64_t* __restrict__ cold, const uint32_t* __restrict__ member_off,
                 const uint16_t* __restrict__ members, double* __restrict__ load, bool lds_ok)
{
    const uint32_t p = blockIdx.x, lane = lane_id();
    const cr_plan_spec spec = specs[p];
    if (!hash_placed(spec.variant)) return;
    const uint32_t A = min((uint32_t)__builtin_amdgcn_readfirstlane((int)num_admitted[p]), Cmax);
    const uint32_t w = min(spec.window, NW - 1u);
    const uint32_t* __restrict__ ocnt = order_count + (uint64_t)w * Cmax;
    const uint32_t* __restrict__ moff = member_off + (uint64_t)p * (Cmax + 1u);
    const uint16_t* __restrict__ mem = members + (uint64_t)p * Cmax;
    const double init = (double)cold[p] / (double)R;
    double Lr[kS];
#pragma unroll
    for (int s = 0; s < kS; ++s) Lr[s] = init;
    // R <= 64 with the plan's lists in LDS (the host gives kS == 1 launches Cmax-sized
    // dynamic LDS when Cmax <= kHashStage): a destination's load needs only its own jobs, in
    // job order. The member copies (job order, each job's members distinct) are sorted
    // stably by destination in LDS, 64 at a time (a copy's rank is its destination's count
    // in earlier chunks plus the earlier lanes of its chunk with the same destination, by
    // ballots over the destination bits); lane r then adds the charges of its own list in
    // order -- the same additions, in the same order per destination, as the job loop below.
    if (kS == 1 && lds_ok) {
        extern __shared__ double s_dyn[];
        double* s_x = s_dyn;                                                  // [Cmax] job charges
        uint16_t* s_mem = reinterpret_cast<uint16_t*>(s_x + Cmax);           // [Cmax] members
        uint16_t* s_job = s_mem + Cmax;                                       // [Cmax] job of a copy
        uint16_t* s_ord = s_job + Cmax;                                       // [Cmax] sorted copies
        uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_ord + Cmax + (Cmax & 1u));  // [64]
        uint32_t* s_run = s_cnt + 64;                                         // [64]
        const uint32_t total = A ? (uint32_t)__builtin_amdgcn_readfirstlane((int)moff[A]) : 0u;  // <= Cmax
        s_cnt[lane] = 0;
        for (uint32_t a = lane; a < A; a += 64u) {
            const uint32_t o = moff[a], k = moff[a + 1u] - o;
            s_x[a] = (double)ocnt[a] / (double)k;
            for (uint32_t t = 0; t < k; ++t) s_job[o + t] = (uint16_t)a;
        }
        for (uint32_t i0 = 0; i0 < total; i0 += 16u * 64u) {  // all loads in flight
            uint32_t v[16];
#pragma unroll
            for (uint32_t u = 0; u < 16; ++u) {
                const uint32_t i = i0 + u * 64u + lane;
                v[u] = i < total ? (uint32_t)mem[i] : 0xFFFFu;
            }
#pragma unroll
            for (uint32_t u = 0; u < 16; ++u) {
                const uint32_t i = i0 + u * 64u + lane;
                if (i < total) {
                    s_mem[i] = (uint16_t)v[u];
                    if (v[u] < R) atomicAdd(&s_cnt[v[u]], 1u);
                }
            }
        }
        __syncthreads();
        const uint32_t cnt = lane < R ? s_cnt[lane] : 0u;
        const uint32_t off = wave_incl_scan_u32(cnt) - cnt;
        s_run[lane] = off;
        __syncthreads();
        uint32_t nbits = 0;
        while ((1u << nbits) < R) ++nbits;
        for (uint32_t i0 = 0; i0 < total; i0 += 64u) {
            const uint32_t i = i0 + lane;
            const uint32_t m = i < total ? (uint32_t)s_mem[i] : 0xFFFFu;
            const bool valid = m < R;
            uint64_t peers = ballot(valid);
            for (uint32_t bit = 0; bit < nbits; ++bit) {
                const bool on = (m >> bit) & 1u;
                const uint64_t bb = ballot(on);
                peers &= on ? bb : ~bb;
            }
            const uint32_t rk = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t at = valid ? s_run[m] + rk : 0u;
            if (valid) s_ord[at] = s_job[i];
            __syncthreads();
            if (valid && rk == 0) s_run[m] = at + (uint32_t)__popcll(peers);
            __syncthreads();
        }
        double L = Lr[0];
        for (uint32_t q = 0; q < cnt; ++q) L = L + s_x[s_ord[off + q]];
        if (lane < R) load[(uint64_t)p * R + lane] = L;
        return;
    }
    for (uint32_t base = 0; base < A; base += 64u) {
        // lane j holds job base + j: its charge, copy count, first member and offset
        const uint32_t a = base + lane;
        double x = 0.0;
        uint32_t k = 0, d = 0xFFFFu, o = 0;
        if (a < A) {
            o = moff[a];
            k = moff[a + 1u] - o;
            x = (double)ocnt[a] / (double)k;
            d = mem[o];
        }
        const uint32_t nb = A - base < 64u ? A - base : 64u;
        for (uint32_t j = 0; j < nb; ++j) {
            const double xj = rdlane_f64(x, j);
            const uint32_t kj = rdlane(k, j);
            if (kj == 1u) {
                const uint32_t dj = rdlane(d, j);
#pragma unroll
                for (int s = 0; s < kS; ++s)
                    if (s * 64u + lane == dj) Lr[s] = Lr[s] + xj;
            } else {
                const uint32_t oj = rdlane(o, j);
                for (uint32_t t = 0; t < kj; ++t) {
                    const uint32_t m = mem[oj + t];
#pragma unroll
                    for (int s = 0; s < kS; ++s)
                        if (s * 64u + lane == m) Lr[s] = Lr[s] + xj;
                }
            }
        }
    }
#pragma unroll
    for (int s = 0; s < kS; ++s) {
        const uint32_t r = s * 64u + lane;
        if (r < R) load[(uint64_t)p * R + r] = Lr[s];
    }
}

// Churn between two plans of a set (Section 5.4; Appendix E, table of replan measurements).
// One block per pair (p, q): its threads walk p's admitted keys in admission order, look
// each key up in q's compact dispatch table (one 16-byte key-index load and a popcount)
// and compare the two member lists; the work per key is k_p * k_q compares.
constexpr uint32_t kChurnThreads = 256;

__global__ void __launch_bounds__(kChurnThreads)
    k_plan_churn(uint32_t NP, uint32_t KW, uint32_t Cmax, uint32_t NW, const cr_plan_spec* __restrict__ specs,
                 const uint32_t* __restrict__ order, const uint32_t* __restrict__ num_admitted,
                 const uint32_t* __restrict__ member_off, const uint16_t* __restrict__ members,
                 const uint64_t* __restrict__ key_index, const uint32_t* __restrict__ route,
                 const uint32_t* __restrict__ pairs, uint64_t* __restrict__ out, uint32_t* __restrict__ err)
{
    __shared__ uint64_t s_acc[4][kChurnThreads / kWave];
    const uint32_t pr = blockIdx.x;
    const uint32_t p = pairs[2u * pr], q = pairs[2u * pr + 1u];
    uint64_t common_pairs = 0, both = 0, k_changed = 0, same_set = 0;
    if (p < NP && q < NP) {
        const uint32_t A = min(num_admitted[p], Cmax);
        const uint32_t w = specs[p].window;
        const uint32_t* ord = order + (uint64_t)min(w, NW - 1u) * Cmax;
        const uint32_t* mop = member_off + (uint64_t)p * (Cmax + 1u);
        const uint16_t* mep = members + (uint64_t)p * Cmax;
        const uint64_t* kxq = key_index + (uint64_t)q * KW * 2u;
        const uint32_t* rwq = route + (uint64_t)q * Cmax;
        const uint32_t* moq = member_off + (uint64_t)q * (Cmax + 1u);
        const uint16_t* meq = members + (uint64_t)q * Cmax;
        for (uint32_t a = w < NW ? threadIdx.x : A; a < A; a += kChurnThreads) {
            const uint32_t b = ord[a];
            const ulonglong2 e = kx_entry(kxq, b, true);
            if (!((e.x >> (b & 63u)) & 1ull)) continue;  // not admitted by q
            const uint32_t word = rwq[kx_rank(e, b)];
            const bool single = (word & CR_ROUTE_SINGLE) != 0u;
            const uint32_t q0 = single ? 0u : moq[word];
            const uint32_t kq = single ? 1u : moq[word + 1u] - q0;
            const uint32_t p0 = mop[a], kp = mop[a + 1u] - p0;
            uint32_t common = 0;
            for (uint32_t i = 0; i < kp; ++i) {
                const uint32_t m = mep[p0 + i];
                if (single) {
                    common += m == (word & 0xFFFFu);
                } else {
                    for (uint32_t t = 0; t < kq; ++t) common += m == (uint32_t)meq[q0 + t];
                }
            }
            common_pairs += common;
            both += 1u;
            k_changed += kp != kq;
            same_set += kp == kq && common == kp;
        }
    } else if (threadIdx.x == 0) {
        atomicOr(err, CR_ERR_SPEC);
    }
    const uint32_t wv = threadIdx.x / kWave;
    common_pairs = wave_sum_u64(common_pairs);
    both = wave_sum_u64(both);
    k_changed = wave_sum_u64(k_changed);
    same_set = wave_sum_u64(same_set);
    if ((threadIdx.x & (kWave - 1u)) == 0u) {
        s_acc[0][wv] = common_pairs;
        s_acc[1][wv] = both;
        s_acc[2][wv] = k_changed;
        s_acc[3][wv] = same_set;
    }
    __syncthreads();
    if (threadIdx.x < 4u) {
        uint64_t v = 0;
#pragma unroll
        for (uint32_t i = 0; i < kChurnThreads / kWave; ++i) v += s_acc[threadIdx.x][i];
        out[4ull * pr + threadIdx.x] = v;
    }
}

inline uint32_t key_words(uint32_t K) { return (K + 63u) / 64u; }

bool valid_set(const cr_plan_set* ps)
{
    if (!ps) return false;
    if (ps->num_plans == 0 || ps->cands == 0 || ps->cands > CR_MAX_CANDS || ps->num_plans % ps->cands) return false;
    if (ps->R == 0 || ps->R > CR_MAX_R || ps->max_W == 0 || ps->max_W > CR_MAX_W) return false;
    if (ps->num_keys == 0 || ps->num_keys == 0xFFFFFFFFu || ps->num_windows == 0) return false;
    if (!ps->specs || !ps->order || !ps->order_count || !ps->n_order || !ps->num_admitted || !ps->cold || !ps->clamped ||
        !ps->member_off || !ps->members || !ps->load || !ps->key_index || !ps->route)
        return false;
    return true;
}

}  // namespace
}  // namespace cr

extern "C" size_t cr_admit_workspace_bytes(uint32_t num_windows, uint32_t R, uint32_t max_W)
{
    const uint64_t cmax = (uint64_t)R * max_W;
    return (size_t)(num_windows * (2u * cmax * sizeof(uint2) + sizeof(uint64_t)) + 256u);
}

extern "C" void cr_plan_sizes(uint32_t num_plans, uint32_t cands, uint32_t R, uint32_t max_W, uint32_t num_keys,
                              uint32_t num_windows, size_t out_bytes[CR_PLAN_BUFFERS])
{
    if (!out_bytes) return;
    const uint64_t NP = num_plans, NW = num_windows, cmax = (uint64_t)R * max_W;
    const uint64_t NG = cands ? NP / cands : 0, CS = ((uint64_t)cands + 7) / 8 * 8;
    const uint64_t KW = ((uint64_t)num_keys + 63) / 64;
    const uint64_t b[CR_PLAN_BUFFERS] = {
        NP * sizeof(cr_plan_spec), NW * cmax * 4, NW * cmax * 4, NW * 4, NP * 4, NP * 8, NP * 4,
        NP * (cmax + 1) * 4, NP * cmax * 2, NP * R * 8, NP * KW * 16, NP * cmax * 4,
        NW * num_keys * 4, NG * cmax * CS * 2, NG * R * CS * 2, NG * cmax * CS * 4};
    for (int i = 0; i < CR_PLAN_BUFFERS; ++i) out_bytes[i] = (size_t)b[i];
}

extern "C" cr_status cr_admit(const uint32_t* counts, const cr_plan_set* plans, void* ws, size_t ws_bytes,
                              uint32_t* err, void* stream)
{
    using namespace cr;
    if (!counts || !valid_set(plans) || !ws || !err) return CR_EINVAL;
    const uint32_t cmax = plans->R * plans->max_W;
    if (ws_bytes < cr_admit_workspace_bytes(plans->num_windows, plans->R, plans->max_W)) return CR_ESIZE;
    uint8_t* base = reinterpret_cast<uint8_t*>(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    uint2* buf = reinterpret_cast<uint2*>(base);
    uint64_t* row_sum = reinterpret_cast<uint64_t*>(base + (uint64_t)plans->num_windows * 2u * cmax * sizeof(uint2));
    const hipStream_t st = as_stream(stream);
    (void)hipGetLastError();
    const uint32_t K = plans->num_keys;
    if (cmax <= kRegCmax && K <= 1024u * 32u) {
#define CR_SORT_REG(NPL)                                                                                            \
    hipLaunchKernelGGL(k_sort_window_reg<NPL>, dim3(plans->num_windows), dim3(kSortBlock), 0, st, counts, K, cmax,  \
                       plans->order, plans->order_count, plans->n_order, row_sum)
        if (K <= 1024u * 4u) CR_SORT_REG(4);
        else if (K <= 1024u * 8u) CR_SORT_REG(8);
        else if (K <= 1024u * 16u) CR_SORT_REG(16);
        else if (K <= 1024u * 20u) CR_SORT_REG(20);
        else CR_SORT_REG(32);
#undef CR_SORT_REG
    } else if (K >= kWideKeys + (uint64_t)kWideKeysPerWindow * plans->num_windows && K <= 0xFFF00000u && cmax >= kWideCmax &&
               plans->num_windows <= kWideWindows) {
        const uint32_t NW = plans->num_windows, tile = wide_tile(K, NW);
        const dim3 tiles((K + tile - 1u) / tile, NW), th(kWideThreads);
        uint32_t *ord = plans->order, *ocnt = plans->order_count;
        hipLaunchKernelGGL(k_wide_zero, dim3(NW), th, 0, st, cmax, ord, ocnt, buf, row_sum);
        hipLaunchKernelGGL(k_wide_hist, tiles, th, 0, st, counts, K, tile, cmax, ord, ocnt, buf, row_sum);
        hipLaunchKernelGGL(k_wide_refine<1>, tiles, th, 0, st, counts, K, tile, cmax, ord, ocnt, buf);
        hipLaunchKernelGGL(k_wide_refine<2>, tiles, th, 0, st, counts, K, tile, cmax, ord, ocnt, buf);
        hipLaunchKernelGGL(k_wide_refine<3>, tiles, th, 0, st, counts, K, tile, cmax, ord, ocnt, buf);
        hipLaunchKernelGGL(k_wide_count, tiles, th, 0, st, counts, K, tile, cmax, ord, ocnt, plans->n_order, buf);
        hipLaunchKernelGGL(k_wide_compact, tiles, th, 0, st, counts, K, tile, cmax, ord, ocnt, buf);
        if (cmax <= kWideSmall) {
            const size_t lds = (size_t)cmax * 16u;
            if (hipFuncSetAttribute((const void*)k_wide_sort, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
                hipSuccess)
                return CR_EHIP;
            hipLaunchKernelGGL(k_wide_sort, dim3(NW), dim3(kSortBlock), lds, st, cmax, ord, ocnt, buf);
        } else {
            const dim3 et((cmax + kWideTile - 1u) / kWideTile, NW);
            for (uint32_t pass = 0; pass < 3u; ++pass) {
                hipLaunchKernelGGL(k_wide_digits, et, th, 0, st, cmax, pass, ord, ocnt, buf);
                hipLaunchKernelGGL(k_wide_offsets, dim3(kWideDigits / 64u, NW), dim3(64), 0, st, cmax, pass, ord, ocnt, buf);
                hipLaunchKernelGGL(k_wide_scatter, et, th, 0, st, cmax, pass, ord, ocnt, buf);
            }
        }
    } else if ((uint64_t)plans->num_keys * 4u <= kSortLdsRowBytes) {
        const uint32_t lds = plans->num_keys * 4u;
        if (hipFuncSetAttribute((const void*)k_sort_window<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return CR_EHIP;
        hipLaunchKernelGGL(k_sort_window<true>, dim3(plans->num_windows), dim3(kSortBlock), (size_t)lds, st, counts,
                           plans->num_keys, cmax, plans->order, plans->order_count, plans->n_order, row_sum, buf);
    } else {
        hipLaunchKernelGGL(k_sort_window<false>, dim3(plans->num_windows), dim3(kSortBlock), 0, st, counts,
                           plans->num_keys, cmax, plans->order, plans->order_count, plans->n_order, row_sum, buf);
    }
    const uint32_t KW = key_words(plans->num_keys);
    const size_t bits = KW <= kKxLdsWords ? (size_t)KW * 8u : 0u;
#define CR_ADMIT(THREADS)                                                                                           \
    do {                                                                                                            \
        if (hipFuncSetAttribute((const void*)k_admit_plan<THREADS>, hipFuncAttributeMaxDynamicSharedMemorySize,      \
                                (int)bits) != hipSuccess)                                                           \
            return CR_EHIP;                                                                                         \
        hipLaunchKernelGGL(k_admit_plan<THREADS>, dim3(plans->num_plans), dim3(THREADS), bits, st, plans->R, cmax,   \
                           plans->num_windows, KW, plans->specs, plans->order, plans->order_count, plans->n_order,   \
                           row_sum, plans->num_admitted, plans->cold, plans->clamped, plans->member_off,             \
                           plans->key_index, err);                                                                   \
    } while (0)
    if ((cmax < plans->num_keys ? cmax : plans->num_keys) <= kAdmitSmall) CR_ADMIT(512);
    else CR_ADMIT(1024);
#undef CR_ADMIT
    return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
}

extern "C" cr_status cr_place_lpt(const uint32_t* counts, const cr_plan_set* plans, void* stream)
{
    using namespace cr;
    if (!counts || !valid_set(plans)) return CR_EINVAL;
    const uint32_t cmax = plans->R * plans->max_W;
    const hipStream_t st = as_stream(stream);
    (void)hipGetLastError();
    if (plans->R <= 64) {
        hipLaunchKernelGGL(k_lpt_small, dim3(plans->num_plans), dim3(64), 0, st, key_words(plans->num_keys), plans->R,
                           cmax, plans->num_windows, plans->specs, plans->order, plans->order_count,
                           plans->num_admitted, plans->cold, plans->member_off, plans->key_index, plans->members,
                           plans->load, plans->route);
        return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
    }
#define CR_LPT_BLOCK(NT)                                                                                          \
    hipLaunchKernelGGL(k_lpt_block<NT>, dim3(plans->num_plans), dim3(NT), 0, st, plans->R, cmax, plans->specs,     \
                       plans->order_count, plans->num_admitted, plans->cold, plans->num_windows, plans->member_off, \
                       plans->members, plans->load)
    if (plans->R <= 128) CR_LPT_BLOCK(128);
    else if (plans->R <= 256) CR_LPT_BLOCK(256);
    else if (plans->R <= 512) CR_LPT_BLOCK(512);
    else CR_LPT_BLOCK(1024);
#undef CR_LPT_BLOCK
    hipLaunchKernelGGL(k_route_words, dim3((cmax + kWordThreads - 1) / kWordThreads, plans->num_plans),
                       dim3(kWordThreads), 0, st, cmax, plans->num_windows, key_words(plans->num_keys), plans->specs,
                       plans->order, plans->num_admitted, plans->member_off, plans->members, plans->key_index,
                       plans->route);
    return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
}

extern "C" cr_status cr_plan_churn(const cr_plan_set* plans, const uint32_t* pairs, uint32_t num_pairs, uint64_t* out,
                                   uint32_t* err, void* stream)
{
    using namespace cr;
    if (!valid_set(plans) || !err || (num_pairs > 0 && (!pairs || !out))) return CR_EINVAL;
    if (num_pairs > 0x7FFFFFFFu) return CR_EINVAL;
    if (num_pairs == 0) return CR_OK;
    const hipStream_t st = as_stream(stream);
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_plan_churn, dim3(num_pairs), dim3(kChurnThreads), 0, st, plans->num_plans,
                       key_words(plans->num_keys), plans->R * plans->max_W, plans->num_windows, plans->specs,
                       plans->order, plans->num_admitted, plans->member_off, plans->members, plans->key_index,
                       plans->route, pairs, out, err);
    return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
}

extern "C" cr_status cr_place_hash(const uint32_t* counts, const cr_plan_set* plans, void* stream)
{
    using namespace cr;
    if (!counts || !valid_set(plans)) return CR_EINVAL;
    const uint32_t cmax = plans->R * plans->max_W;
    const hipStream_t st = as_stream(stream);
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_hash_members, dim3(plans->num_plans, (cmax + kHashThreads - 1) / kHashThreads),
                       dim3(kHashThreads), 0, st, plans->R, cmax, plans->num_windows, key_words(plans->num_keys),
                       plans->specs, plans->order, plans->num_admitted, plans->member_off, plans->key_index,
                       plans->members, plans->route);
#define CR_HASH_LOADS(S, LDS, OK)                                                                                   \
    hipLaunchKernelGGL(k_hash_loads<S>, dim3(plans->num_plans), dim3(64), (LDS), st, plans->R, cmax,                  \
                       plans->num_windows, plans->specs, plans->order_count, plans->num_admitted, plans->cold,        \
                       plans->member_off, plans->members, plans->load, (OK))
    const uint32_t s = (plans->R + 63) / 64;
    const bool lds_ok = s <= 1 && cmax <= kHashStage;  // R <= 64: the plan's lists fit in LDS
    if (s <= 1) CR_HASH_LOADS(1, lds_ok ? hash_loads_lds_bytes(cmax) : 0, lds_ok);
    else if (s <= 2) CR_HASH_LOADS(2, 0, false);
    else if (s <= 4) CR_HASH_LOADS(4, 0, false);
    else if (s <= 8) CR_HASH_LOADS(8, 0, false);
    else CR_HASH_LOADS(16, 0, false);
#undef CR_HASH_LOADS
    return hipGetLastError() == hipSuccess ? CR_OK : CR_EHIP;
}

// ---------------------------------------------------------------------------------------
// cr_admit_noalloc: cr_admit with its workspace in a library-owned device array instead of
// the caller's. The array is a file-scope __device__ variable; its name in host code is a
// stand-in, so its device address is taken once per device with hipGetSymbolAddress (with
// that device current) and kept. Every call on a device shares that device's array.
// ---------------------------------------------------------------------------------------
namespace cr {
namespace {

constexpr size_t kAdmitScratchBytes = (size_t)CR_ADMIT_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) uint8_t scratch[kAdmitScratchBytes];

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];

cr_status admit_scratch(void** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CR_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CR_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return CR_OK;
}

}  // namespace
}  // namespace cr

extern "C" cr_status cr_admit_noalloc(const uint32_t* counts, const cr_plan_set* plans, uint32_t* err, void* stream)
{
    using namespace cr;
    if (!counts || !valid_set(plans) || !err) return CR_EINVAL;
    if (cr_admit_workspace_bytes(plans->num_windows, plans->R, plans->max_W) > kAdmitScratchBytes) return CR_ESIZE;
    void* ws = nullptr;
    const cr_status st = admit_scratch(&ws);
    if (st != CR_OK) return st;
    return cr_admit(counts, plans, ws, kAdmitScratchBytes, err, stream);
}
