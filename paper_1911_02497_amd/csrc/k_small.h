// Bin searches of one wavefront in an LDS histogram, and the rest of a ranking on a short list by one workgroup.
#pragma once
#include "k_select.h"

namespace condensa {

constexpr u64 kSmallCallElems = static_cast<u64>(1) << 21;
constexpr int kSmallFinishThreads = 1024;

// Wavefront 0 of a workgroup: the bin of an LDS histogram (nb <= kBins bins) that holds descending rank r, i.e.
// #(keys in higher bins) < r <= #(keys in bins >= bin).  The lane that finds it writes bin, the rank inside
// the bin, the bin's count and *found = 1; nothing is written when the histogram holds fewer than r keys.
__device__ inline void wave_pick_desc(const u32* s_hist, int nb, u64 r, u32* bin, u64* rem, u64* cnt, u32* found) {
    constexpr int kPerMax = kBins / 64;
    const int lane = threadIdx.x & 63;
    const int per = (nb + 63) / 64;
    u32 c[kPerMax];
    u64 sum = 0;
#pragma unroll
    for (int i = 0; i < kPerMax; ++i) {
        const int b = nb - 1 - (lane * per + i);
        c[i] = (i < per && b >= 0) ? s_hist[b] : 0u;
        sum += c[i];
    }
    const u64 incl = wave_incl_scan_u64(sum);
    u64 before = incl - sum;
    if (before < r && r <= incl) {
#pragma unroll
        for (int i = 0; i < kPerMax; ++i) {
            if (before < r && r <= before + c[i]) {
                *bin = static_cast<u32>(nb - 1 - (lane * per + i));
                *rem = r - before;
                *cnt = c[i];
                *found = 1u;
            }
            before += c[i];
        }
    }
}

// The same for ascending rank r (the r-th lowest), used for the index search among ties.
__device__ inline void wave_pick_asc(const u32* s_hist, int nb, u64 r, u32* bin, u64* rem, u32* found) {
    constexpr int kPerMax = kBins / 64;
    const int lane = threadIdx.x & 63;
    const int per = (nb + 63) / 64;
    u32 c[kPerMax];
    u64 sum = 0;
#pragma unroll
    for (int i = 0; i < kPerMax; ++i) {
        const int b = lane * per + i;
        c[i] = (i < per && b < nb) ? s_hist[b] : 0u;
        sum += c[i];
    }
    const u64 incl = wave_incl_scan_u64(sum);
    u64 before = incl - sum;
    if (before < r && r <= incl) {
#pragma unroll
        for (int i = 0; i < kPerMax; ++i) {
            if (before < r && r <= before + c[i]) {
                *bin = static_cast<u32>(lane * per + i);
                *rem = r - before;
                *found = 1u;
            }
            before += c[i];
        }
    }
}

// A 1024-thread workgroup finishes one ranking on a list of (key, index) entries that holds every key sharing the
// ranking's digits above `first_level` (and possibly other keys): `e` is the ranking's state on entering that
// level.  The remaining levels are counted in LDS over the matching entries, the tie rule picks the r-th lowest
// index among the entries equal to the threshold, and the outcome becomes the ranking's stored state and its
// result record.  Called by every thread of the workgroup with the same arguments.
template <typename KEY, typename IDX>
__device__ inline void finish_on_list(Slot& slot, SlotStep e, const KEY* __restrict__ keys, const IDX* __restrict__ ids,
                                      u64 n_list, int key_bits, int first_level, int idx_bits, condensa_select* record) {
    __shared__ __align__(8) u32 s_hist[kBins];
    __shared__ u32 s_bin, s_found, s_n;
    __shared__ u64 s_rem, s_cnt;
    const int tid = threadIdx.x;
    u64 tie_end = slot.n;                                  // every tie kept, unless found otherwise below
    if (e.state == kSelecting) {                           // uniform over the workgroup
        u64 prefix = e.prefix, r = e.remaining, n_tie = 0;
        bool ok = true;
        for (int level = first_level; level < n_levels(key_bits) && ok; ++level) {
            const Level lv = level_of(key_bits, level);
            const int nb = 1 << lv.bits;
            for (int i = tid; i < nb; i += kSmallFinishThreads) s_hist[i] = 0;
            if (tid == 0) s_found = 0;
            __syncthreads();
            for (u64 i = tid; i < n_list; i += kSmallFinishThreads) {
                const u64 key = keys[i];
                if (((key ^ prefix) >> lv.hi_shift) == 0) atomicAdd(&s_hist[static_cast<u32>(key >> lv.shift) & (nb - 1)], 1u);
            }
            __syncthreads();
            if (tid < 64) wave_pick_desc(s_hist, nb, r, &s_bin, &s_rem, &s_cnt, &s_found);
            __syncthreads();
            ok = s_found != 0;
            if (ok) {
                prefix |= static_cast<u64>(s_bin) << lv.shift;
                r = s_rem;
                n_tie = s_cnt;
            }
            __syncthreads();
        }
        if (!ok) {
            e.state = kFailed;                             // the counts of the levels and the list disagree: reported, not hidden
        } else {
            e.prefix = prefix; e.remaining = r; e.n_tie = n_tie; e.state = kDone; e.need_tie = 0;
            const u64 T = prefix;
            if (r < n_tie && n_tie <= static_cast<u64>(kSmallFinishThreads)) {
                // a handful of ties: their indices in LDS, each ranked by counting the lower ones
                u64* s_idx = reinterpret_cast<u64*>(s_hist);
                if (tid == 0) { s_n = 0; s_rem = slot.n - 1; }
                __syncthreads();
                for (u64 i = tid; i < n_list; i += kSmallFinishThreads)
                    if (static_cast<u64>(keys[i]) == T) {
                        const u32 p = atomicAdd(&s_n, 1u);
                        if (p < static_cast<u32>(kSmallFinishThreads)) s_idx[p] = static_cast<u64>(ids[i]);
                    }
                __syncthreads();
                const u32 m = s_n < static_cast<u32>(kSmallFinishThreads) ? s_n : static_cast<u32>(kSmallFinishThreads);
                if (static_cast<u32>(tid) < m) {
                    const u64 mine = s_idx[tid];
                    u64 lower = 0;
                    for (u32 i = 0; i < m; ++i) lower += (s_idx[i] < mine) ? 1u : 0u;
                    if (lower + 1 == r) s_rem = mine;      // indices are distinct: one thread
                }
                __syncthreads();
                tie_end = s_rem + 1;
            } else if (r < n_tie) {
                // many ties: radix levels on the index over the entries equal to the threshold, lowest first
                u64 iprefix = 0, ir = r;
                for (int level = 0; level < n_levels(idx_bits); ++level) {     // uniform
                    const Level lv = level_of(idx_bits, level);
                    const int nb = 1 << lv.bits;
                    for (int i = tid; i < nb; i += kSmallFinishThreads) s_hist[i] = 0;
                    if (tid == 0) s_found = 0;
                    __syncthreads();
                    for (u64 i = tid; i < n_list; i += kSmallFinishThreads) {
                        if (static_cast<u64>(keys[i]) != T) continue;
                        const u64 idx = static_cast<u64>(ids[i]);
                        if (((idx ^ iprefix) >> lv.hi_shift) == 0) atomicAdd(&s_hist[static_cast<u32>(idx >> lv.shift) & (nb - 1)], 1u);
                    }
                    __syncthreads();
                    if (tid < 64) wave_pick_asc(s_hist, nb, ir, &s_bin, &s_rem, &s_found);
                    __syncthreads();
                    iprefix |= static_cast<u64>(s_bin) << lv.shift;
                    ir = s_rem;
                    __syncthreads();
                }
                tie_end = iprefix + 1;
            }
        }
    }
    if (tid != 0) return;
    if (slot.state == kSelecting) {
        slot.prefix = e.prefix; slot.remaining = e.remaining; slot.n_tie = e.n_tie;
        slot.state = e.state; slot.need_tie = 0;
        slot.tie_end = tie_end;
    }
    condensa_select out;
    out.n = slot.n;
    out.k = slot.k;
    if (e.state == kDone) {
        out.n_gt = slot.k - e.remaining;
        out.n_tie_kept = e.remaining;
        out.n_tie = e.n_tie;
        out.threshold_key = e.prefix;
        out.tie_end = slot.tie_end;
    } else {                                               // k == 0: nothing is kept
        out.n_gt = 0; out.n_tie_kept = 0; out.n_tie = 0;
        out.threshold_key = ~static_cast<u64>(0);
        out.tie_end = 0;
    }
    out.path = slot.path;
    *record = out;
}

}  // namespace condensa
