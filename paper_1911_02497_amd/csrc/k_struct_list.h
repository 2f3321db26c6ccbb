// Structure rankings of moderate size (more than k_struct_small's 4096 structures, at most kSmallCallElems, GLOBAL
// scope): one histogram over a window of the aggregates, then a list.  Filters, neurons, blocks in place, of more than 256 elements or of
// more than two dimensions; other blocks go in strips (k_struct_strip.h).
//
// The six levels of a 63-bit ranking are six dependent launches plus the tie search, and the first of them separate little:
// aggregates of one model share their sign and most exponent bits.  So every workgroup of k_struct_list_hist first takes the
// same 256 aggregates and bounds the threshold by two of their order statistics, six standard deviations of its rank to
// either side; 2047 equal steps between them are the bins, and what lies outside belongs to the first or last one.
// k_struct_list_collect lists the (key, id) pairs of the threshold's bin, a hundred or so, and k_struct_list_finish, one
// workgroup, finishes on the list.  The list can hold every structure, so nothing overflows, and a sample that misleads
// makes it longer, never wrong.  A long list is equal aggregates as a rule, and those at its ends are found without ranking
// it (2^20 blocks of 4x4, nine tenths of them pruned before: 1812 us ranked, 120 now).  Two radix levels instead of the
// window took 13 + 11 us for a Transformer's 688 128 blocks of 8x8 and 12 + 10 for 270 400 blocks of 5x5; this one 11.4 and
// 8.2.
// Table 1 (FilterPrune, BlockPrune: structures are aggregated and pruned); Section 3.1.
#pragma once
#include "k_small.h"
#include "k_structure.h"
#include "k_window.h"

namespace condensa {

constexpr u32 kStructSample = 256;        // aggregates of the sample, one per thread

struct StructListArgs {
    u64* count;            // entries offered (never more than cap: the list holds every structure)
    u64* key;              // [cap]
    u32* id;               // [cap] global structure ids
    u64 cap;
    u32* window;           // its lower end (upper halves of the keys) and the shift of its bins
    struct StructPiece* piece;       // [F / kKeyPiece, rounded up] of a long list: what each piece of the aggregates adds to it
};
struct StructPiece {
    u64 least, most;       // of its listed keys (none: ~0 and 0)
    u32 n_least, n_most;   // how many are equal to these
};
constexpr u32 kListHeld = 4096;           // list entries held in LDS; a list with more is long
constexpr u64 kMaxPieces = kSmallCallElems / kKeyPiece;
static_assert(kMaxPieces <= kSmallFinishThreads && kKeyPiece == 2 * kSmallFinishThreads, "k_struct_list_finish: a thread a piece, two keys a thread");

__device__ inline u32 struct_window_bin(u64 key, u32 lo, u32 shift) {
    const u32 hi = static_cast<u32>(key >> 32);
    const u32 b = hi < lo ? 0u : (hi - lo) >> shift;
    return b < static_cast<u32>(kBins) ? b : static_cast<u32>(kBins) - 1u;
}

// The bin of the threshold: the histogram stands where that of radix level 0 would, whose digit has as many values.
__device__ inline SlotStep struct_window_step(const StructArgs& a, u32* bin) {
    const SlotStep e = wave_enter_level(a.slots[0], 1, 63, struct_hist(a, 0), struct_coarse(a, 0));
    *bin = static_cast<u32>(e.prefix >> level_of(63, 0).shift);
    return e;
}
static_assert(kBins == 1 << 11, "radix level 0 of 63 bits has 11 bits");

__global__ __launch_bounds__(kBlock) void k_struct_list_hist(StructArgs a, StructListArgs l, u64 pieces_per_block) {
    static_assert(kStructSample == kBlock, "one sampled aggregate per thread");
    __shared__ __align__(16) u32 s_hist[kBins];
    __shared__ u32 s_sample[kStructSample];
    __shared__ u32 s_end[2];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const Slot& slot = a.slots[0];
    if (slot_canonical(slot).state != kSelecting) return;  // uniform: k == 0, nothing to rank
    // one from each of as many equal stretches, at a place of its own in it: evenly spaced ones can all lie in one column of
    // blocks (every 1024th or 4096th of a matrix whose rows of blocks are powers of two), whose scale need not be the others'
    const u64 place = (static_cast<u64>(tid) * a.F + __umul64hi(static_cast<u64>(mix32(tid + 1)) << 32, a.F)) / kStructSample;
    s_sample[tid] = static_cast<u32>(a.keys[place] >> 32);
    for (int i = tid; i < kBins; i += kBlock) s_hist[i] = 0;
    __syncthreads();
    if (wave < 2) {                                        // wavefront 0: the upper end, 1: the lower end
        const double p = static_cast<double>(slot.k) / static_cast<double>(a.F), S = kStructSample;
        const double off = 6.0 * sqrt(S * p * (1.0 - p)) + 2.0, at = p * S + (wave == 0 ? -off : off);
        const u32 want = at < 1.0 ? 1u : (at > S ? kStructSample : static_cast<u32>(at));
        u32 v[4], found = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = s_sample[lane + 64 * i];
        for (int bit = 30; bit >= 0; --bit) {              // the want-th largest, bit by bit
            const u32 c = found | (1u << bit);
            u32 n = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) n += __popcll(__ballot(v[i] >= c));
            if (n >= want) found = c;
        }
        if (found == 0 && wave == 1) {                     // zeros (weights pruned before): a window from there on would leave
            u32 least = 0xFFFFFFFFu;                       // a bin half an octave wide; what lies four octaves below the least
#pragma unroll                                             // sampled value goes with the zeros
            for (int i = 0; i < 4; ++i) least = v[i] != 0 && v[i] < least ? v[i] : least;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) { const u32 o = __shfl_xor(least, d, 64); least = o < least ? o : least; }
            if (least != 0xFFFFFFFFu && least > (4u << 20)) found = least - (4u << 20);
        }
        if (lane == 0) s_end[wave] = found;
    }
    __syncthreads();
    const u32 hi = s_end[0], lo = s_end[1] < hi ? s_end[1] : hi, span = hi - lo;
    const u32 shift = span < static_cast<u32>(kBins) ? 0u : 21u - static_cast<u32>(__clz(static_cast<int>(span)));
    if (blockIdx.x == 0 && tid == 0) { l.window[0] = lo; l.window[1] = shift; }
    const u64 base = static_cast<u64>(blockIdx.x) * pieces_per_block * kKeyPiece;
    const u64 stop = base + pieces_per_block * kKeyPiece < a.F ? base + pieces_per_block * kKeyPiece : a.F;
    for (u64 i0 = base + tid; i0 < stop; i0 += kKeyPiece) {
        constexpr int kPer = static_cast<int>(kKeyPiece) / kBlock;
        u64 key[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const u64 i = i0 + static_cast<u64>(u) * kBlock;
            key[u] = i < stop ? a.keys[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (i0 + static_cast<u64>(u) * kBlock < stop) atomicAdd(&s_hist[struct_window_bin(key[u], lo, shift)], 1u);
    }
    __syncthreads();
    u64* hist = struct_hist(a, 0);
    for (int i = tid; i < kBins; i += kBlock) {
        const u32 v = s_hist[i];
        if (v) atomicAdd(reinterpret_cast<unsigned long long*>(hist + i), static_cast<unsigned long long>(v));
    }
    static_assert(kBins / kCoarse == 32 && kBins / kBlock == 8, "four threads add up the bins of a coarse sum");
    const uint4 x = *reinterpret_cast<const uint4*>(s_hist + 8 * tid), y = *reinterpret_cast<const uint4*>(s_hist + 8 * tid + 4);
    u32 sum = x.x + x.y + x.z + x.w + y.x + y.y + y.z + y.w;
    sum += __shfl_xor(sum, 1, 64);
    sum += __shfl_xor(sum, 2, 64);
    if ((tid & 3u) == 0 && sum)
        atomicAdd(reinterpret_cast<unsigned long long*>(struct_coarse(a, 0) + tid / 4), static_cast<unsigned long long>(sum));
}

__global__ __launch_bounds__(kBlock) void k_struct_list_collect(StructArgs a, StructListArgs l) {
    __shared__ u32 s_bin, s_selecting, s_long;
    __shared__ u64 s_wave[kBlock / 64];
    __shared__ u64 s_base;
    __shared__ StructPiece s_piece;
    const int tid = threadIdx.x;
    if (tid < 64) {
        u32 bin;
        const SlotStep e = struct_window_step(a, &bin);
        if (tid == 0) { s_bin = bin; s_selecting = e.state == kSelecting ? 1u : 0u; s_long = e.n_tie > kListHeld ? 1u : 0u; }
    }
    __syncthreads();
    if (s_selecting == 0) return;                          // uniform: k == 0, nothing to rank
    const u32 bin = s_bin, lo = l.window[0], shift = l.window[1];
    for (u64 base = static_cast<u64>(blockIdx.x) * kKeyPiece; base < a.F; base += static_cast<u64>(gridDim.x) * kKeyPiece) {
        const u64 end = (base + kKeyPiece < a.F) ? base + kKeyPiece : a.F;
        const u64* __restrict__ kp = a.keys;               // the ranking is over all structures: their keys are one array
        constexpr int kPer = static_cast<int>(kKeyPiece) / kBlock;             // keys per thread, strided by the workgroup
        u64 key[kPer];
        u32 listed = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const u64 i = base + tid + static_cast<u64>(u) * kBlock;
            key[u] = (i < end) ? kp[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (base + tid + static_cast<u64>(u) * kBlock < end && struct_window_bin(key[u], lo, shift) == bin) listed |= 1u << u;
        u64 total;
        const u64 before = block_excl_scan_u64(static_cast<u64>(__popc(listed)), s_wave, &total);
        if (s_long) {                                      // uniform
            if (tid == 0) s_piece = StructPiece{~static_cast<u64>(0), 0, 0, 0};
            __syncthreads();
            u64 least = ~static_cast<u64>(0), most = 0;
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (listed & (1u << u)) { least = key[u] < least ? key[u] : least; most = key[u] > most ? key[u] : most; }
            if (listed) {
                atomicMin(reinterpret_cast<unsigned long long*>(&s_piece.least), static_cast<unsigned long long>(least));
                atomicMax(reinterpret_cast<unsigned long long*>(&s_piece.most), static_cast<unsigned long long>(most));
            }
            __syncthreads();
            u32 n_least = 0, n_most = 0;
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (listed & (1u << u)) { n_least += key[u] == s_piece.least ? 1u : 0u; n_most += key[u] == s_piece.most ? 1u : 0u; }
            if (n_least) atomicAdd(&s_piece.n_least, n_least);
            if (n_most) atomicAdd(&s_piece.n_most, n_most);
            __syncthreads();
            if (tid == 0) l.piece[base / kKeyPiece] = s_piece;
        }
        if (total != 0) {                                  // uniform over the workgroup
            if (tid == 0) s_base = atomicAdd(reinterpret_cast<unsigned long long*>(l.count), static_cast<unsigned long long>(total));
            __syncthreads();
            u64 pos = s_base + before;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                if (listed & (1u << u)) {
                    if (pos < l.cap) {
                        l.key[pos] = key[u];
                        l.id[pos] = static_cast<u32>(base + tid + static_cast<u64>(u) * kBlock);
                    }
                    ++pos;
                }
            }
            __syncthreads();                               // s_base is rewritten for the next chunk
        }
    }
}


// One workgroup ranks the list, applies the lowest-id rule among equal aggregates and writes state and record.  A lone
// workgroup is bound by latency: four radix levels over a list in memory took 22 us for the 688 128 blocks, one level of
// eight bits and pairs in LDS 5.9.
__global__ __launch_bounds__(kSmallFinishThreads) void k_struct_list_finish(StructArgs a, StructListArgs l, condensa_select* results,
                                                                           int id_bits) {
    __shared__ SlotStep s_e;
    __shared__ RankShared sh;
    __shared__ u64 s_key[kListHeld];
    __shared__ u32 s_tie[kSmallFinishThreads];
    __shared__ u32 s_n;
    __shared__ u64 s_last;
    __shared__ StructPiece s_ends;
    __shared__ u32 s_wave[kSmallFinishThreads / 64], s_at[2];
    Slot& slot = a.slots[0];
    const u32 tid = threadIdx.x;
    u64 n64 = *l.count;
    if (n64 > l.cap) n64 = l.cap;                          // (cannot happen: the list holds every structure)
    const u32 n = static_cast<u32>(n64);
    const bool held = n <= kListHeld;
    if (held) for (u32 i = tid; i < n; i += kSmallFinishThreads) s_key[i] = l.key[i];
    if (tid == 0) s_n = 0;
    if (tid < 64) {
        u32 bin;
        const SlotStep e = struct_window_step(a, &bin);
        if (tid == 0) s_e = e;
    }
    __syncthreads();
    SlotStep e = s_e;
    u64 tie_end = slot.n;                                  // every tie kept, unless found otherwise below
    if (e.state == kSelecting) {                           // uniform
        auto key_of = [&](u32 i) { return held ? s_key[i] : l.key[i]; };
        // A long list is ties as a rule (blocks pruned before), at one end of it: then nothing in it needs to be ranked.  The
        // pieces say how many there are and, one after the other, where the last one kept lies.
        bool at_end = false;
        if (!held) {                                       // uniform
            const u32 pieces = static_cast<u32>((a.F + kKeyPiece - 1) / kKeyPiece);
            const StructPiece mine = tid < pieces ? l.piece[tid] : StructPiece{~static_cast<u64>(0), 0, 0, 0};
            if (tid == 0) s_ends = StructPiece{~static_cast<u64>(0), 0, 0, 0};
            __syncthreads();
            atomicMin(reinterpret_cast<unsigned long long*>(&s_ends.least), static_cast<unsigned long long>(mine.least));
            atomicMax(reinterpret_cast<unsigned long long*>(&s_ends.most), static_cast<unsigned long long>(mine.most));
            __syncthreads();
            const u32 n_least = mine.least == s_ends.least ? mine.n_least : 0u, n_most = mine.most == s_ends.most ? mine.n_most : 0u;
            if (n_least) atomicAdd(&s_ends.n_least, n_least);
            if (n_most) atomicAdd(&s_ends.n_most, n_most);
            __syncthreads();
            const u32 r = static_cast<u32>(e.remaining), beyond = n - s_ends.n_least;          // keys above the least one
            const bool top = r <= s_ends.n_most;
            at_end = top || r > beyond;
            if (at_end) {                                  // uniform
                const u64 T = top ? s_ends.most : s_ends.least;
                const u32 rank = top ? r : r - beyond, ties = top ? s_ends.n_most : s_ends.n_least, here = top ? n_most : n_least;
                e.prefix = T; e.remaining = rank; e.n_tie = ties; e.state = kDone; e.need_tie = 0;
                if (rank < ties) {
                    u32 total;
                    const u32 upto = wg_incl_scan_u32<kSmallFinishThreads>(here, s_wave, &total);
                    if (upto - here < rank && rank <= upto) { s_at[0] = tid; s_at[1] = rank - (upto - here); }
                    __syncthreads();
                    const u64 i0 = s_at[0] * kKeyPiece + 2 * tid;
                    const u32 e0 = i0 < a.F && a.keys[i0] == T ? 1u : 0u, e1 = i0 + 1 < a.F && a.keys[i0 + 1] == T ? 1u : 0u;
                    const u32 before = wg_incl_scan_u32<kSmallFinishThreads>(e0 + e1, s_wave, &total) - e0 - e1, want = s_at[1];
                    if (before < want && want <= before + e0 + e1) s_last = i0 + (e0 && want == before + 1 ? 0 : 1);
                    __syncthreads();
                    tie_end = s_last + 1;
                }
            }
        }
        if (at_end) {
        } else if (!rank_keys<kSmallFinishThreads>(sh, n, key_of, e.remaining)) {
            e.state = kFailed;                             // the counts of the levels and the list disagree: reported, not hidden
        } else {
            const u64 T = sh.key, r = sh.rem;
            e.prefix = T; e.remaining = r; e.n_tie = sh.n_tie; e.state = kDone; e.need_tie = 0;
            if (r < e.n_tie && e.n_tie <= static_cast<u64>(kSmallFinishThreads)) {
                // their ids in LDS, each ranked by counting the lower ones
                for (u32 i = tid; i < n; i += kSmallFinishThreads)
                    if (key_of(i) == T) s_tie[atomicAdd(&s_n, 1u)] = l.id[i];
                __syncthreads();
                const u32 m = static_cast<u32>(e.n_tie);
                if (tid < m) {
                    const u32 mine = s_tie[tid];
                    u32 lower = 0;
                    for (u32 i = 0; i < m; ++i) lower += (s_tie[i] < mine) ? 1u : 0u;
                    if (lower + 1 == r) s_last = mine;     // ids are distinct: one thread
                }
                __syncthreads();
                tie_end = s_last + 1;
            } else if (r < e.n_tie) {
                // many ties: radix levels on the id over the entries equal to the threshold, lowest first
                u64 iprefix = 0, ir = r;
                for (int level = 0; level < n_levels(id_bits); ++level) {      // uniform
                    const Level lv = level_of(id_bits, level);
                    const int nb = 1 << lv.bits;
                    for (int i = tid; i < nb; i += kSmallFinishThreads) sh.hist[i] = 0;
                    __syncthreads();
                    for (u32 i = tid; i < n; i += kSmallFinishThreads) {
                        if (key_of(i) != T) continue;
                        const u64 idx = l.id[i];
                        if (((idx ^ iprefix) >> lv.hi_shift) == 0) atomicAdd(&sh.hist[static_cast<u32>(idx >> lv.shift) & (nb - 1)], 1u);
                    }
                    __syncthreads();
                    if (tid < 64) wave_pick_asc(sh.hist, nb, ir, &sh.bin, &sh.rem, &sh.found);
                    __syncthreads();
                    iprefix |= static_cast<u64>(sh.bin) << lv.shift;
                    ir = sh.rem;
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
    const bool done = e.state == kDone;                    // else k == 0: nothing is kept
    out.n = slot.n;
    out.k = slot.k;
    out.n_gt = done ? slot.k - e.remaining : 0;
    out.n_tie_kept = done ? e.remaining : 0;
    out.n_tie = done ? e.n_tie : 0;
    out.threshold_key = done ? e.prefix : ~static_cast<u64>(0);
    out.tie_end = done ? slot.tie_end : 0;
    out.path = slot.path;
    *results = out;
}

}  // namespace condensa
