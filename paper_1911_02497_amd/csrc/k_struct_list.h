// Structure rankings of moderate size (more than k_struct_small's 4096 structures, at most kSmallCallElems, GLOBAL
// scope): two radix levels over the aggregates, then a list.
//
// The six levels of a 63-bit ranking are six dependent launches plus the tie search.  Aggregates of one model share
// their sign and most exponent bits, so level 0 barely separates them; after level 1 (22 of 63 bits) the threshold's
// bin holds a few hundred structures.  k_struct_list_collect lists those (key, structure id) pairs and
// k_struct_list_finish, one workgroup, finishes on the list.  The list can hold every structure, so nothing overflows.  A Transformer's 688 128 blocks of 8x8: 14 -> 10 launches.
// Table 1 (FilterPrune, BlockPrune: structures are aggregated and pruned); Section 3.1.
#pragma once
#include "k_small.h"
#include "k_structure.h"

namespace condensa {

constexpr int kStructListLevels = 2;      // radix levels counted over all aggregates before the list takes over

struct StructListArgs {
    u64* count;            // entries offered (never more than cap: the list holds every structure)
    u64* key;              // [cap]
    u32* id;               // [cap] global structure ids
    u64 cap;
};

__global__ __launch_bounds__(kBlock) void k_struct_list_collect(StructArgs a, StructListArgs l) {
    __shared__ SlotStep s_e;
    __shared__ u64 s_wave[kBlock / 64];
    __shared__ u64 s_base;
    const int tid = threadIdx.x;
    if (tid < 64) {
        const SlotStep e = wave_enter_level(a.slots[0], kStructListLevels, 63, struct_hist(a, kStructListLevels - 1),
                                            struct_coarse(a, kStructListLevels - 1));
        if (tid == 0) s_e = e;
    }
    __syncthreads();
    if (s_e.state != kSelecting) return;                   // uniform: k == 0, nothing to rank
    const u64 prefix = s_e.prefix;
    const Level L = level_of(63, kStructListLevels - 1);   // entries agree with the prefix down to this level's digit
    for (u64 base = static_cast<u64>(blockIdx.x) * kKeyPiece; base < a.F; base += static_cast<u64>(gridDim.x) * kKeyPiece) {
        const u64 end = (base + kKeyPiece < a.F) ? base + kKeyPiece : a.F;
        const u64* __restrict__ kp = a.keys;               // the ranking is over all structures: their keys are one array
        constexpr int kPer = static_cast<int>(kKeyPiece) / kBlock;             // keys per thread, strided by the workgroup
        u64 key[kPer];
        u32 listed = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const u64 i = base + tid + static_cast<u64>(u) * kBlock;
            key[u] = (i < end) ? kp[i] : ~prefix;          // a filler that fails the prefix test
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (base + tid + static_cast<u64>(u) * kBlock < end && ((key[u] ^ prefix) >> L.shift) == 0) listed |= 1u << u;
        u64 total;
        const u64 before = block_excl_scan_u64(static_cast<u64>(__popc(listed)), s_wave, &total);
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

constexpr u32 kListHeld = 4096;           // list entries held in LDS

// One workgroup ranks the list, applies the lowest-id rule among equal aggregates and writes state and record.  A lone
// workgroup is bound by latency: four more levels over a list in memory took 22 us for the 688 128 blocks, one level
// and pairs in LDS 5.9.
__global__ __launch_bounds__(kSmallFinishThreads) void k_struct_list_finish(StructArgs a, StructListArgs l, condensa_select* results,
                                                                           int id_bits) {
    __shared__ SlotStep s_e;
    __shared__ RankShared sh;
    __shared__ u64 s_key[kListHeld];
    __shared__ u32 s_tie[kSmallFinishThreads];
    __shared__ u32 s_n;
    __shared__ u64 s_last;
    Slot& slot = a.slots[0];
    const u32 tid = threadIdx.x;
    u64 n64 = *l.count;
    if (n64 > l.cap) n64 = l.cap;                          // (cannot happen: the list holds every structure)
    const u32 n = static_cast<u32>(n64);
    const bool held = n <= kListHeld;
    if (held) for (u32 i = tid; i < n; i += kSmallFinishThreads) s_key[i] = l.key[i];
    if (tid == 0) s_n = 0;
    if (tid < 64) {
        const SlotStep e = wave_enter_level(slot, kStructListLevels, 63, struct_hist(a, kStructListLevels - 1),
                                            struct_coarse(a, kStructListLevels - 1));
        if (tid == 0) s_e = e;
    }
    __syncthreads();
    SlotStep e = s_e;
    u64 tie_end = slot.n;                                  // every tie kept, unless found otherwise below
    if (e.state == kSelecting) {                           // uniform
        auto key_of = [&](u32 i) { return held ? s_key[i] : l.key[i]; };
        if (!rank_keys<kSmallFinishThreads>(sh, n, key_of, e.remaining)) {
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
