// Bin searches of one wavefront in an LDS histogram, and the rest of a ranking on a short list by one workgroup.
#pragma once
#include "k_select.h"

namespace condensa {

constexpr u64 kSmallCallElems = static_cast<u64>(1) << 21;
constexpr int kSmallFinishThreads = 1024;

// Wavefront 0 of a workgroup: the bin of an LDS histogram (nb <= kBins bins) that holds ascending rank r (the r-th lowest), used for
// the index search among ties.  The lane that finds it writes bin, the rank inside the bin and *found = 1; nothing is written when
// the histogram holds fewer than r keys.
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

// Ranking of n keys of at most 63 bits by one workgroup.  Radix levels of eight bits from the highest bit in which the keys
// differ (aggregates of one model share their sign and most exponent bits), until at most kRankPairs share the digits
// found; those are ranked by comparing all pairs, four threads to a key.  A lone workgroup is bound by latency: one search
// of 2048 bins takes a wavefront 3.7 us, one of 256 bins 0.5 and its counts 0.6; 255 keys in pairs take 3.2 us (64-bit
// compares are quarter rate), 64 keys 0.8.
constexpr u32 kRankPairs = 64;
struct RankShared {
    __align__(16) u32 hist[kBins];                         // rank_keys uses the first 256
    u64 pair[kRankPairs];
    u32 any, all;          // OR and AND of the keys' upper halves
    u64 key, rem, n_tie;   // result: the key at the rank, how many of its equals are kept, how many there are
    u32 n, bin, found;
};

// sh.key = the key at descending rank `rank` (1-based) of key_of(0..n-1), sh.rem, sh.n_tie; false when there are fewer.
// Every thread of the THREADS (at least 4 kRankPairs) calls it and gets the same value; it ends with a barrier.
template <int THREADS, typename KeyOf>
__device__ inline bool rank_keys(RankShared& sh, u32 n, KeyOf key_of, u64 rank64) {
    static_assert(THREADS >= 4 * static_cast<int>(kRankPairs), "four threads to a key");
    const u32 tid = threadIdx.x;
    u32 any = 0, all = ~0u;
    for (u32 i = tid; i < n; i += THREADS) { const u32 hi = static_cast<u32>(key_of(i) >> 32); any |= hi; all &= hi; }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { any |= __shfl_xor(any, d, 64); all &= __shfl_xor(all, d, 64); }
    if (tid == 0) { sh.any = 0; sh.all = ~0u; sh.found = (rank64 >= 1 && rank64 <= n) ? 1u : 0u; }
    if (tid < 256) sh.hist[tid] = 0;
    __syncthreads();
    if ((tid & 63u) == 0) {
        atomicOr(&sh.any, any);
        atomicAnd(&sh.all, all);
    }
    __syncthreads();
    if (sh.found == 0) return false;                       // uniform
    const u32 diff = sh.any ^ sh.all;
    int top = diff == 0 ? 32 : 64 - __clz(static_cast<int>(diff));             // bits below which the keys may differ
    u64 prefix = ((static_cast<u64>(sh.all) << 32) >> top) << top;
    if (diff == 0 && n > kRankPairs) {                     // uniform: the same for the lower halves (ties above all)
        any = 0; all = ~0u;
        for (u32 i = tid; i < n; i += THREADS) { const u32 low = static_cast<u32>(key_of(i)); any |= low; all &= low; }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) { any |= __shfl_xor(any, d, 64); all &= __shfl_xor(all, d, 64); }
        __syncthreads();
        if (tid == 0) { sh.any = 0; sh.all = ~0u; }
        __syncthreads();
        if ((tid & 63u) == 0) { atomicOr(&sh.any, any); atomicAnd(&sh.all, all); }
        __syncthreads();
        const u32 low_diff = sh.any ^ sh.all;
        top = low_diff == 0 ? 0 : 32 - __clz(static_cast<int>(low_diff));
        prefix |= (static_cast<u64>(sh.all) >> top) << top;
    }
    u32 rank = static_cast<u32>(rank64), n_in = n;
    while (top > 0 && n_in > kRankPairs) {                 // uniform; the 256 counts are clear here
        const int bits = top < 8 ? top : 8, shift = top - bits;
        const u32 mask = (1u << bits) - 1u;
        for (u32 i = tid; i < n; i += THREADS) {
            const u64 key = key_of(i);
            if (((key ^ prefix) >> top) == 0) atomicAdd(&sh.hist[static_cast<u32>(key >> shift) & mask], 1u);
        }
        __syncthreads();
        if (tid < 64) {                                    // four bins a lane, from the top
            const uint4 c4 = *reinterpret_cast<const uint4*>(sh.hist + 252 - 4 * tid);
            const u32 c[4] = {c4.w, c4.z, c4.y, c4.x};
            u32 before = wave_incl_scan_u32(c[0] + c[1] + c[2] + c[3]) - (c[0] + c[1] + c[2] + c[3]);
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
                if (before < rank && rank <= before + c[i]) { sh.bin = 255 - 4 * tid - i; sh.rem = rank - before; sh.n = c[i]; }
                before += c[i];
            }
        }
        __syncthreads();
        if (tid < 256) sh.hist[tid] = 0;
        prefix |= static_cast<u64>(sh.bin) << shift;
        rank = static_cast<u32>(sh.rem);
        n_in = sh.n;
        top = shift;
        __syncthreads();
    }
    if (top == 0) {
        if (tid == 0) { sh.key = prefix; sh.rem = rank; sh.n_tie = n_in; }
    } else {
        if (tid == 0) sh.n = 0;
        __syncthreads();
        for (u32 i = tid; i < n; i += THREADS) {
            const u64 key = key_of(i);
            if (((key ^ prefix) >> top) == 0) sh.pair[atomicAdd(&sh.n, 1u)] = key;        // n_in of them
        }
        __syncthreads();
        const u32 mine = tid >> 2;
        if (tid < 4 * kRankPairs) {                        // whole wavefronts: the lanes of a key trade their counts
            const u64 key = sh.pair[mine < n_in ? mine : 0];
            u32 higher = 0, same = 0;
#pragma unroll 8
            for (u32 e = tid & 3u; e < n_in; e += 4) {
                const u64 k2 = sh.pair[e];
                higher += k2 > key ? 1u : 0u;
                same += k2 == key ? 1u : 0u;
            }
            higher += __shfl_xor(higher, 1, 64); same += __shfl_xor(same, 1, 64);
            higher += __shfl_xor(higher, 2, 64); same += __shfl_xor(same, 2, 64);
            if (mine < n_in && higher < rank && rank <= higher + same) {       // equals write the same
                sh.key = key; sh.rem = rank - higher; sh.n_tie = same;
            }
        }
    }
    __syncthreads();
    return true;
}

}  // namespace condensa
