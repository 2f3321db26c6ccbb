// BlockPrune (Table 1) with the weights read once: 2-D blocks of any size up to kStripArea elements, GLOBAL scope, three launches.
//
// Aggregates first and then an apply sweep read the weights twice, with five small launches in between (13 bytes a weight and some
// 30 us).  Here, as in k_struct_fused.h and k_listed.h, a sample supplies a prior and results never depend on it:
//   1. k_strip_begin fetches the tables, clears, and in the same launch samples: every sampling workgroup ranks the aggregates
//      of its own blocks and leaves the keys at the threshold's expected rank, from which list_bounds takes a window [lo, hi] on the
//      aggregates' upper 31 bits and an estimate `mid`.
//   2. k_struct_strips: a workgroup takes a strip of blocks -- a piece of a row of blocks, or several whole rows of them in
//      a narrow matrix -- into LDS with coalesced loads, a thread adds up each block in memory order, and the strip leaves again
//      from the registers it was loaded into: theta and mask are final outside the window, provisional inside (kept from `mid` on).  The blocks
//      inside are counted in equal bins over the window, and their keys and ids go into a few places that each bin has.
//   3. k_strip_resolve: every workgroup finds the threshold's bin and ranks what lies there, some ten blocks, for itself; nobody waits for
//      anybody.  Then it settles its own strips: structure mask, kept ids (the strips' provisional counts, corrected by what lies
//      between estimate and threshold, say how many come before) and the few blocks that were decided wrongly.
//      Where the window missed, or a bin has more than its places (equal aggregates), the workgroups that are running find the threshold
//      in a few passes over the stored keys, meeting in between (Meet), and settle in the same way.
// Against aggregates, list and apply sweep, us a call: 688 128 blocks of 8x8 in 96 matrices 134 -> 98 (traced: 9, 77 and 16), 270 400 of 5x5 51.6 -> 39
// (9, 18 and 13), 786 thousand of 4x4 69 -> 49, 172 thousand of 16x16 122 -> 101, 2.7 M of 5x5 304 -> 203, 16.8 M of 4x4 890 -> 669.
// Weights pruned before (2^20 blocks of 4x4, nine tenths of them zero, the threshold among them) 114 -> 87.  Slower where windows hold a gap: two scales in any order with the
// threshold between them 74.4 -> 82.4, halves 74.6 -> 79.7, a quarter of blocks of which half are larger 78.6 -> 87.2, half of the blocks that are not zero 80.8 -> 82.7.
// Section 3.1 (the schemes aggregate blocks), Table 1 (BlockPrune: blocks of any dimensionality and a given size).
#pragma once
#include "k_listed.h"
#include "k_structure.h"

namespace condensa {

constexpr int kStripThreads = 128;               // of the sweep
constexpr int kResolveThreads = 512;
constexpr u32 kStripSettle = kResolveThreads * 4;          // blocks that a workgroup settles at a time
constexpr int kStripBegin = 512;                 // threads of the launch that begins the call
constexpr u32 kStripPer = 4;                     // loads of four elements that a thread makes for half a strip
constexpr u32 kStripQuads = kStripPer * kStripThreads;
constexpr u32 kStripLds = 2304;                  // elements of half a strip in LDS (sixteen workgroups would fit into a compute unit's)
constexpr u32 kStripBlocks = 2 * kStripThreads;  // blocks of a strip at most
constexpr u32 kStripArea = 256;                  // elements of a block at most: the chain of additions of one thread
constexpr u32 kStripCopies = 4;                  // counters of a bin, chosen by strip
constexpr u32 kStripMostSlots = 1024;            // places of a bin at most, the same number for each counter
constexpr u32 kStripMostBins = 2048;             // every workgroup of k_strip_resolve reads all counters (with 8192 bins, 2.7 M blocks took it 86 us)
constexpr u32 kStripGather = 256;                // blocks that the fallback ranks by all pairs at most (836 took 110 us, a pass over 16.8 M keys 37)
static_assert(kStripGather <= kStripMostSlots);
constexpr u32 kStripAboves = 64;                 // counters of the blocks above the window, a line each
constexpr u32 kStripTensors = 1024;              // tensors of a call at most: a wavefront looks at all their starts
constexpr u32 kStripLanes = 4, kStripSample = kStripBegin / kStripLanes;           // lanes that share a sampled block, and blocks of a workgroup at once
constexpr u32 kStripRounds = 2;                  // at most
constexpr int kStripPassBits = 10;
constexpr u32 kStripPassBins = 1u << kStripPassBits;
constexpr u32 kStripPassWords = kStripPassBins * 5 + kListLine;          // counts, greatest and (complemented) least keys, and the keys above
constexpr int kStripResolveGrid = 512;           // two to a compute unit

struct StripArgs {
    const ListWin* win;
    u32* hist;             // [bins][kStripCopies] blocks offered
    u64* key;              // [bins][kStripCopies][room]
    u32* id;
    u32 log_bins;          // at least 8
    u32 log_room;          // at least 5
    u32 log_group;         // strips whose counts are added up, a power of two
    u32 n_tiles;
    u32* above;            // [kStripAboves][kListLine]
    uint2* tiles;          // [n_tiles + 1] first id and provisionally kept blocks of a strip
    u32* coarse;           // [n_tiles / group + 1][kListLine] the latter added up, a line each: the updates of a line take turns, some 10 ns each
    u32* pass;             // [3][kStripPassWords] a pass of the fallback: this one, the next and the one being cleared
    u32* meet;             // [kMeetWords]
    u32* share;            // [2][kStripResolveGrid] keys above the threshold and ties in the share of each workgroup
    u64* tie_end;
    const OutDesc* out;
    int32_t* keep_idx;
    u8* user_mask;
    condensa_select* results;
    int quad;              // every access to the tensors takes sixteen bytes, aligned, inside one block
    u32 units;             // quads, or elements, of a block
    FastDiv by_units;
};

// A tensor's strips, in the spare words of its descriptor: the first one's number, block columns and block rows of a strip (several rows of
// whole width, or one) and strips across.
__host__ __device__ inline u32 strip_start(const TensorDesc& d) { return static_cast<u32>(d.reserved[0]); }
__host__ __device__ inline u32 strip_across(const TensorDesc& d) { return static_cast<u32>(d.reserved[0] >> 32); }
__host__ __device__ inline u32 strip_down(const TensorDesc& d) { return static_cast<u32>(d.reserved[1]); }
__host__ __device__ inline u32 strips_across(const TensorDesc& d) { return static_cast<u32>(d.reserved[1] >> 32); }

// Lays the strips of a matrix of d2 x d3 in blocks of b2 x b3 (at most kStripArea elements together); `first` is the number of the first
// one.  As many block columns as fit, in pieces of equal width, then as many rows of blocks.  Returns how many strips there are.
inline u64 strip_layout(TensorDesc* d, bool quad, u64 first) {
    const u64 d2 = d->d[2], d3 = d->d[3], b2 = d->b[2], b3 = d->b[3], G2 = (d2 + b2 - 1) / b2, G3 = (d3 + b3 - 1) / b3;
    const u64 stride = quad ? b3 : b3 | 1;                 // of a block's column in LDS: odd, so that neighbours' banks differ
    auto fits = [&](u64 across, u64 down) {
        const u64 cols = across * b3 < d3 ? across * b3 : d3, half = (down * b2 + 1) / 2;
        return across * down <= kStripBlocks && half * across * stride <= kStripLds && half * ((cols + 3) / 4) <= kStripQuads;
    };
    u64 across = G3 < kStripBlocks ? G3 : kStripBlocks;
    while (across > 1 && !fits(across, 1)) --across;
    const u64 pieces = (G3 + across - 1) / across;
    across = (G3 + pieces - 1) / pieces;
    if (quad && pieces > 1) {                              // whole lines of 128 bytes, so that no two strips write to one
        u64 lines = 1;
        while (lines * b3 % 32 != 0) lines *= 2;
        const u64 up = (across + lines - 1) / lines * lines;
        if (fits(up, 1)) across = up;
    }
    const u64 pieces_now = (G3 + across - 1) / across;
    u64 down = 1;
    while (pieces_now == 1 && down < G2 && fits(across, down + 1)) ++down;
    const u64 rows = (G2 + down - 1) / down;
    down = (G2 + rows - 1) / rows;
    d->reserved[0] = first | (across << 32);
    d->reserved[1] = down | (pieces_now << 32);
    return rows * pieces_now;
}

// Bins over the window, and from where on a block is provisionally kept: of a crowded window's equals, none.
__device__ inline u32 strip_shift(const ListWin& w, u32 log_bins) {
    const u32 span = w.hi - w.lo;
    return span < (1u << log_bins) ? 0u : 32u - log_bins - static_cast<u32>(__clz(static_cast<int>(span)));
}
__device__ inline u32 strip_mid(const ListWin& w) { return win_crowded(w) ? w.hi + 1u : w.mid; }
// Where the draws say that the keys crowd at a few places (equal ones, a gap), too many would meet in a bin: a few of its places are no use,
// and its counters would be what the sweep waits for (2^20 blocks of 4x4 in two scales, the threshold between them: 127 us
// listed, 82 now).
__device__ inline bool strip_listed(const ListWin& w) { return !win_crowded(w) && !win_uneven(w); }

// ---- sample ----------------------------------------------------------------------------------------------

struct StripMatrix { const float* w; u32 start, d2, d3; };

// One sampling workgroup, number `me` of W (a power of two): kStripSample ROUNDS blocks out of as many equal stretches of the population, in units of
// four neighbours (which share lines), four lanes to a block (one lane alone made up to 32 loads of single elements, each from another line: the
// launch took 19.7 us for 270 400 blocks of 5x5).  Bound by latency.  Their sums are added in any order and in binary32: a sample need not be exact (blocks
// of 16x16: 10.5 us, in binary64 16.5).  Blocks whose squares leave binary32 (weights below 1e-22 or beyond 1e19) lie outside every window, then, and the fallback
// takes them.
template <typename MatrixOf>
__device__ inline void strip_sample(const ListArgs& w, u32 W, u32 me, u32 rounds, u32 b2, u32 b3, int quad, u64 F, u64 k, MatrixOf&& matrix_of) {
    __shared__ __align__(16) u32 s_key[kStripRounds * kStripSample];
    const u32 tid = threadIdx.x, mine = tid % kStripLanes, count = rounds * kStripSample;
    for (u32 i = tid / kStripLanes; i < count; i += kStripSample) {      // uniform
        const u32 units = static_cast<u32>(F / 4), turn = mix32(~(i >> 2)) & (W - 1);      // every W-th stretch can lie in one column of blocks, whose scale
        const u32 u = (i >> 2) * W + ((me + turn) & (W - 1));                            // is its own
        const int log_stretches = 31 - __clz(static_cast<int>(count / 4 * W));
        const u32 place = static_cast<u32>((static_cast<u64>(u) * units + __umulhi(mix32(u), units)) >> log_stretches);
        const u64 id = static_cast<u64>(place < units ? place : units - 1) * 4 + (i & 3u);
        const StripMatrix m = matrix_of(id);
        const u32 G3 = (m.d3 + b3 - 1) / b3, s = static_cast<u32>(id - m.start), g2 = s / G3, g3 = s - g2 * G3;
        const u32 h = m.d2 - g2 * b2 < b2 ? m.d2 - g2 * b2 : b2, wd = m.d3 - g3 * b3 < b3 ? m.d3 - g3 * b3 : b3;
        const float* p = m.w + static_cast<u64>(g2) * b2 * m.d3 + static_cast<u64>(g3) * b3;
        const u32 per = quad ? 4u : 1u, n = h * wd / per, in_row = wd / per, inv = ((1u << 20) + in_row - 1) / in_row;
        float acc = 0.0f;
        for (u32 j0 = 0; j0 < b2 * b3 / per; j0 += 8 * kStripLanes) {     // uniform; every lane loads, without a branch
            float4 v[8];
#pragma unroll
            for (u32 j = 0; j < 8; ++j) {
                const u32 e = j0 + j * kStripLanes + mine, c = e < n ? e : 0, row = (c * inv) >> 20;
                const float* const q = p + static_cast<u64>(row) * m.d3 + (c - row * in_row) * per;
                if (quad) v[j] = *reinterpret_cast<const float4*>(q);
                else      v[j] = make_float4(*q, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (u32 j = 0; j < 8; ++j) {
                const float x = v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
                acc += j0 + j * kStripLanes + mine < n ? x : 0.0f;
            }
        }
#pragma unroll
        for (u32 d = 1; d < kStripLanes; d *= 2) acc += __shfl_xor(acc, static_cast<int>(d), 64);
        if (mine == 0) s_key[i] = static_cast<u32>(static_cast<u64>(__double_as_longlong(static_cast<double>(acc))) >> 32) & 0x7FFFFFFFu;
    }
    __syncthreads();
    // every key's rank by counting, four threads to a key; the three wanted ranks as in list_sample_units, one to either side
    const float all = static_cast<float>(count), ks = static_cast<float>(k) / static_cast<float>(F) * all;
    const u64 tag = static_cast<u64>(w.tag) << 32;
    for (u32 i = tid / kStripLanes; i < count; i += kStripSample) {      // uniform
        const u32 key = s_key[i];
        u32 higher = 0, same = 0, lower = 0;                   // lower: equal ones before this
#pragma unroll 8
        for (u32 e0 = 0; e0 < count; e0 += 4 * kStripLanes) {
            const u32 e = e0 + 4 * mine;
            const uint4 x = *reinterpret_cast<const uint4*>(s_key + e);
            higher += (x.x > key ? 1u : 0u) + (x.y > key ? 1u : 0u) + (x.z > key ? 1u : 0u) + (x.w > key ? 1u : 0u);
            same += (x.x == key ? 1u : 0u) + (x.y == key ? 1u : 0u) + (x.z == key ? 1u : 0u) + (x.w == key ? 1u : 0u);
            lower += (x.x == key && e < i ? 1u : 0u) + (x.y == key && e + 1 < i ? 1u : 0u) + (x.z == key && e + 2 < i ? 1u : 0u) + (x.w == key && e + 3 < i ? 1u : 0u);
        }
#pragma unroll
        for (u32 d = 1; d < kStripLanes; d *= 2) {
            higher += __shfl_xor(higher, static_cast<int>(d), 64);
            same += __shfl_xor(same, static_cast<int>(d), 64);
            lower += __shfl_xor(lower, static_cast<int>(d), 64);
        }
#pragma unroll
        for (u32 which = 0; which < 3; ++which) {
            float x = which == 0 ? floorf(ks - 1.0f) : (which == 1 ? ceilf(ks + 1.0f) + 1.0f : floorf(ks + 0.5f));
            if (which == 2) x = x < 1.0f ? 1.0f : (x > all ? all : x);
            const u32 want = x >= 1.0f && x <= all ? static_cast<u32>(x) : 0u;
            u64* const to = &w.local[static_cast<u64>(which) * w.n_local + me];
            if (want == 0) { if (tid == 0) st_dev64(to, tag | kSampleNone); }
            // so many of a hundred equal: their bins would have no room for them, and their counters no time
            else if (mine == 0 && lower == 0 && higher < want && want <= higher + same) st_dev64(to, tag | key | (same >= 4 && same * 64 >= count ? kListCrowded : 0u));
        }
    }
}

constexpr int kStripBeginTensors = 96;
struct StripBeginArgs {
    UploadArgs up;
    uint4* zero;
    u64 n_zero;            // 16-byte words
    u64 F, k;
    int n_tensors;
    u32 groups;            // sampling workgroups: after the one that fetches the tables
    u32 fillers;           // workgroups that clear: after these.  Then one that bounds the window
    u32 rounds;            // of samples in each
    u32 b2, b3;
    int quad;
    const float* w[kStripBeginTensors];
    u32 start[kStripBeginTensors + 1];
    u32 d2[kStripBeginTensors], d3[kStripBeginTensors];
};
static_assert(sizeof(StripBeginArgs) + sizeof(ListArgs) <= 3584, "kernel arguments");

__global__ __launch_bounds__(kStripBegin) void k_strip_begin(StripBeginArgs b, ListArgs w) {
    const u32 tid = threadIdx.x;
    if (blockIdx.x == 0) {
        upload_words(b.up, tid, kStripBegin);
        __syncthreads();                                   // every load has returned: its value went into a store
        if (tid == 0) store_ticket(b.up.done, b.up.ticket);
        return;
    }
    const u32 block = blockIdx.x - 1;
    if (block >= b.groups + b.fillers) {                   // from what the workgroups before it leave
        list_bounds<true, false, 0u>(w, 1, 0, 0, b.groups, [](u32) { return false; });
        return;
    }
    if (block < b.groups) {
        __shared__ StripMatrix s_m[kStripBeginTensors];
        if (tid < static_cast<u32>(b.n_tensors)) s_m[tid] = StripMatrix{b.w[tid], b.start[tid], b.d2[tid], b.d3[tid]};
        __syncthreads();
        strip_sample(w, b.groups, block, b.rounds, b.b2, b.b3, b.quad, b.F, b.k, [&](u64 id) {
            int lo = 0, hi = b.n_tensors - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_m[mid].start <= id) lo = mid; else hi = mid - 1;
            }
            return s_m[lo];
        });
        return;
    }
    const uint4 z = make_uint4(0, 0, 0, 0);
    for (u64 i = static_cast<u64>(block - b.groups) * kStripBegin + tid; i < b.n_zero; i += static_cast<u64>(b.fillers) * kStripBegin) b.zero[i] = z;
}

// The same as launches of their own (many tensors, captured calls).
__global__ __launch_bounds__(kStripBegin) void k_strip_sample(StructArgs a, ListArgs w, u32 rounds, u32 b2, u32 b3, int quad) {
    strip_sample(w, gridDim.x, blockIdx.x, rounds, b2, b3, quad, a.F, a.slots[0].k, [&](u64 id) {
        const TensorDesc& td = a.td[tensor_of_struct(a.td, a.n_tensors, id)];
        return StripMatrix{td.w, static_cast<u32>(td.struct_start), td.d[2], td.d[3]};
    });
}
__global__ __launch_bounds__(64) void k_strip_bounds(ListArgs w, u32 groups) { list_bounds<false, false, 0u>(w, 1, 0, 0, groups, [](u32) { return false; }); }

// ---- the sweep ---------------------------------------------------------------------------------------------

typedef float f32x4_loose __attribute__((ext_vector_type(4), aligned(4)));
typedef u32 u32_loose __attribute__((aligned(1)));

// QUAD: widths and rows are multiples of four elements and everything is aligned, so that four elements that are loaded together belong to one
// block; in LDS the quads of a block change places so that sixteen neighbouring blocks lie in different banks.  Otherwise: four elements of a row
// at any alignment, the last four of a piece of a row ending with it (some elements twice, the same values); neighbouring blocks stand an odd number of
// words apart in LDS.
// Bound by memory, once enough is under way: a strip takes some 15 us from its first load to its last store, so what a compute unit holds decides.  All of
// a strip's loads are in flight at once, but only half of its rows stand in LDS at a time (the sums go on from the first half to the second).  The
// registers (90 and 91) let ten workgroups onto a compute unit, 160 KB of weights.
template <bool QUAD>
__global__ __launch_bounds__(kStripThreads, 5) void k_struct_strips(StructArgs a, StripArgs s, double* sumsq, float* norms) {
    __shared__ __align__(16) float s_tile[kStripLds];
    __shared__ u8 s_keep[kStripBlocks];
    __shared__ u32 s_count[2];
    constexpr u32 kMine = kStripBlocks / kStripThreads;    // blocks that a thread adds up at most
    const u32 tid = threadIdx.x, lane = tid & 63u, tile = blockIdx.x;
    u32 upto = 0;                                          // tensors whose first strip is not beyond this one: uniform
    for (u32 t0 = 0; t0 < static_cast<u32>(a.n_tensors); t0 += 64) {
        const u32 i = t0 + lane;
        upto += static_cast<u32>(__popcll(__ballot(i < static_cast<u32>(a.n_tensors) && strip_start(a.td[i < static_cast<u32>(a.n_tensors) ? i : 0]) <= tile)));
    }
    const TensorDesc& td = a.td[upto - 1];
    const OutDesc o = s.out[upto - 1];
    const ListWin win = *s.win;
    const u32 d2 = td.d[2], d3 = td.d[3], b2 = td.b[2], b3 = td.b[3];
    const FastDiv by_b2 = td.fd[kDivB2], by_b3 = td.fd[kDivB3];
    const u32 G3 = fast_div(d3 + b3 - 1, by_b3), G2 = fast_div(d2 + b2 - 1, by_b2);
    const u32 number = tile - strip_start(td), pieces = strips_across(td), down_most = strip_down(td), across_most = strip_across(td);
    const u32 at2 = pieces == 1 ? number : number / pieces, g2 = at2 * down_most, g3 = pieces == 1 ? 0u : (number - at2 * pieces) * across_most;
    const u32 down = G2 - g2 < down_most ? G2 - g2 : down_most, across = G3 - g3 < across_most ? G3 - g3 : across_most;
    const u32 r0 = g2 * b2, c0 = g3 * b3, rows = d2 - r0 < down * b2 ? d2 - r0 : down * b2, cols = d3 - c0 < across * b3 ? d3 - c0 : across * b3;
    const u32 n_blocks = down * across, half = (rows + 1) / 2;
    const u64 origin = static_cast<u64>(r0) * d3 + c0, u0 = td.struct_start + static_cast<u64>(g2) * G3 + g3;
    const u32 in_row = (cols + 3) / 4, recip = 0xFFFFFFFFu / in_row + 1;
    const u32 stride = QUAD ? b3 : b3 | 1u, lds_row = across * stride;
    const u32 per_block = b3 / 4, log_per = 31u - static_cast<u32>(__clz(static_cast<int>(per_block | 1u)));
    const u32 swap_mask = (per_block & (per_block - 1)) ? 0u : per_block - 1, swap_shift = log_per < 4 ? 4 - log_per : 0u;      // (QUAD)
    const float* const w = td.w + origin;
    const bool narrow = !QUAD && cols < 4, plain = !QUAD && !narrow && stride == b3;       // uniform

    float4 v[2 * kStripPer];
    u32 where[2 * kStripPer];                              // row << 16 | column
#pragma unroll
    for (u32 i = 0; i < 2 * kStripPer; ++i) {
        const bool second = i >= kStripPer;
        const u32 first_row = second ? half : 0u, n_quads = (second ? rows - half : half) * in_row;
        u32 q = (second ? i - kStripPer : i) * kStripThreads + tid;
        q = q < n_quads ? q : 0u;                          // every lane loads, without a branch
        u32 row = in_row == 1 ? q : __umulhi(q, recip);
        u32 col = (q - row * in_row) * 4;
        if (!QUAD && !narrow) col = col < cols - 4 ? col : cols - 4;
        row = row + first_row < rows ? row + first_row : 0u;             // (a second half without rows)
        where[i] = row << 16 | col;
        const float* p = w + static_cast<u64>(row) * d3 + col;
        if (QUAD) {
            v[i] = ld4_stream(p);
        } else if (!narrow) {
            const f32x4_loose x = __builtin_nontemporal_load(reinterpret_cast<const f32x4_loose*>(p));
            v[i] = make_float4(x.x, x.y, x.z, x.w);
        } else {
            v[i] = make_float4(p[0], cols > 1 ? p[cols > 1 ? 1 : 0] : 0.0f, cols > 2 ? p[cols > 2 ? 2 : 0] : 0.0f, 0.0f);
        }
    }
    if (tid == 0) { s_count[0] = 0; s_count[1] = 0; }
    const u32 b0 = (tid + 64 * (tile & 1u)) & (kStripThreads - 1);       // the first block that this thread adds up
    double acc[kMine];
    u32 br_of[kMine], bc_of[kMine];
#pragma unroll
    for (u32 g = 0; g < kMine; ++g) {
        const u32 b = b0 + g * kStripThreads, bb = b < n_blocks ? b : 0u;
        acc[g] = 0.0;
        br_of[g] = down == 1 ? 0u : bb / across;
        bc_of[g] = bb - br_of[g] * across;
    }
#pragma unroll
    for (u32 part = 0; part < 2; ++part) {
        const u32 p0 = part == 0 ? 0u : half, p1 = part == 0 ? half : rows, n_quads = (p1 - p0) * in_row;
        if (part == 1) __syncthreads();                    // the first half is added up
#pragma unroll
        for (u32 j = 0; j < kStripPer; ++j) {
            const u32 i = part * kStripPer + j;
            if (j * kStripThreads + tid >= n_quads) continue;
            const u32 row = (where[i] >> 16) - p0, col = where[i] & 0xFFFFu;
            const u32 bc = fast_div(col, by_b3);
            u32 x = col - bc * b3;
            if constexpr (QUAD) {
                const u32 at = row * (lds_row / 4) + bc * per_block + ((x / 4) ^ ((bc >> swap_shift) & swap_mask));
                reinterpret_cast<float4*>(s_tile)[at] = v[i];
            } else {
                u32 at = row * lds_row + bc * stride + x;
                if (plain) {                               // uniform: what a column is away from another it is in LDS too
                    s_tile[at] = v[i].x; s_tile[at + 1] = v[i].y; s_tile[at + 2] = v[i].z; s_tile[at + 3] = v[i].w;
                } else {
                    const float e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                    for (u32 k = 0; k < 4; ++k) {
                        if (k < cols) s_tile[at] = e[k];
                        ++at;
                        if (++x == b3) { x = 0; at += stride - b3; }
                    }
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (u32 g = 0; g < kMine; ++g) {
            if (((b0 + g * kStripThreads) & ~63u) >= n_blocks) continue;               // uniform over the wavefront
            const u32 from = br_of[g] * b2 > p0 ? br_of[g] * b2 : p0, block_end = (br_of[g] + 1) * b2, to = block_end < p1 ? block_end : p1;
            const u32 h = to > from ? to - from : 0u, wd = cols - bc_of[g] * b3 < b3 ? cols - bc_of[g] * b3 : b3;
            if (h == 0) continue;
            double sum = acc[g];
            if constexpr (QUAD) {
                const float4* const base = reinterpret_cast<const float4*>(s_tile) + (from - p0) * (lds_row / 4) + bc_of[g] * per_block;
                const u32 turn = (bc_of[g] >> swap_shift) & swap_mask, wq = wd / 4, n = h * wq;
                u32 x = 0, at = 0;
                auto next = [&]() {
                    const float4 t = base[at + (x ^ turn)];
                    if (++x == wq) { x = 0; at += lds_row / 4; }
                    return t;
                };
                float4 t0 = next(), t1 = t0;
                if (n > 1) t1 = next();
                for (u32 i = 0; i + 2 < n; ++i) {          // two quads ahead
                    const float4 t2 = next();
                    sum = add_squares(sum, t0);
                    t0 = t1;
                    t1 = t2;
                }
                sum = add_squares(sum, t0);
                if (n > 1) sum = add_squares(sum, t1);
            } else {
                const float* row = s_tile + (from - p0) * lds_row + bc_of[g] * stride;
                for (u32 r = 0; r < h; ++r, row += lds_row) {
                    u32 x = 0;
                    for (; x + 4 <= wd; x += 4) {
                        float t[4];
#pragma unroll
                        for (u32 k = 0; k < 4; ++k) t[k] = row[x + k];
#pragma unroll
                        for (u32 k = 0; k < 4; ++k) { const double y = static_cast<double>(t[k]); sum = sum + y * y; }
                    }
                    for (; x < wd; ++x) { const double y = static_cast<double>(row[x]); sum = sum + y * y; }
                }
            }
            acc[g] = sum;
        }
    }
    u64 key[kMine];
    u32 list_at[kMine], place[kMine];
    const u32 room = 1u << s.log_room;
#pragma unroll
    for (u32 g = 0; g < kMine; ++g) {
        const u32 b = b0 + g * kStripThreads;
        place[g] = room;
        key[g] = 0;
        list_at[g] = 0;
        if ((b & ~63u) >= n_blocks) continue;              // uniform over the wavefront
        const bool mine = b < n_blocks;
        key[g] = static_cast<u64>(__double_as_longlong(acc[g])) & 0x7FFFFFFFFFFFFFFFull;
        const u32 upper = static_cast<u32>(key[g] >> 32);
        const bool keep = mine && upper >= strip_mid(win);
        const u64 kept = __ballot(keep), beyond = __ballot(mine && upper > win.hi);
        if (lane == 0) {
            if (kept) atomicAdd(&s_count[0], static_cast<u32>(__popcll(kept)));
            if (beyond) atomicAdd(&s_count[1], static_cast<u32>(__popcll(beyond)));
        }
        s_keep[b] = keep ? 1 : 0;
        if (mine) {
            if (strip_listed(win) && upper - win.lo <= win.hi - win.lo) {
                list_at[g] = ((upper - win.lo) >> strip_shift(win, s.log_bins)) * kStripCopies + tile % kStripCopies;
                place[g] = atomicAdd(&s.hist[list_at[g]], 1u);           // on its way while the strip is written
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        s.tiles[tile] = make_uint2(static_cast<u32>(u0), s_count[0]);
        if (s_count[0]) atomicAdd(&s.coarse[(tile >> s.log_group) * kListLine], s_count[0]);
        if (s_count[1]) atomicAdd(&s.above[tile % kStripAboves * kListLine], s_count[1]);
        if (tile + 1 == s.n_tiles) s.tiles[s.n_tiles] = make_uint2(static_cast<u32>(a.F), 0u);
    }
    float* const th = o.theta ? o.theta + origin : nullptr;
    u8* const mk = o.mask ? o.mask + origin : nullptr;
#pragma unroll
    for (u32 i = 0; i < 2 * kStripPer; ++i) {
        const bool second = i >= kStripPer;
        if ((second ? i - kStripPer : i) * kStripThreads + tid >= (second ? rows - half : half) * in_row) continue;
        const u32 row = where[i] >> 16, col = where[i] & 0xFFFFu;
        const u64 e = static_cast<u64>(row) * d3 + col;
        const u32 bc = fast_div(col, by_b3);
        u32 at = (down == 1 ? 0u : fast_div(row, by_b2) * across) + bc;
        if (QUAD) {
            const u8 k = s_keep[at];
            if (th) st4_stream(th + e, k ? v[i].x : 0.0f, k ? v[i].y : 0.0f, k ? v[i].z : 0.0f, k ? v[i].w : 0.0f);
            if (mk) st_mask4_stream(mk + e, k, k, k, k);
        } else {
            u32 x = col - bc * b3, m = 0;                  // mask bytes
            if (b3 >= 3 && !narrow) {                      // uniform: four elements lie in two blocks at most
                const u32 end = b3 - x, in_first = end >= 4 ? 0xFFFFFFFFu : (1u << (8 * end)) - 1u;
                m = (s_keep[at] * 0x01010101u & in_first) | (s_keep[end >= 4 ? at : at + 1] * 0x01010101u & ~in_first);
            } else {
#pragma unroll
                for (u32 j = 0; j < 4; ++j) {
                    m |= (j < cols ? static_cast<u32>(s_keep[at]) : 0u) << (8 * j);
                    if (++x == b3) { x = 0; ++at; }
                }
            }
            auto kept = [&](float y, u32 j) { return (m >> (8 * j)) & 1u ? y : 0.0f; };
            if (!narrow) {
                if (th) {
                    f32x4_loose t;
                    t.x = kept(v[i].x, 0); t.y = kept(v[i].y, 1); t.z = kept(v[i].z, 2); t.w = kept(v[i].w, 3);
                    __builtin_nontemporal_store(t, reinterpret_cast<f32x4_loose*>(th + e));
                }
                if (mk) *reinterpret_cast<u32_loose*>(mk + e) = m;
            } else {
                for (u32 j = 0; j < cols; ++j) {
                    if (th) th[e + j] = j == 0 ? kept(v[i].x, 0) : (j == 1 ? kept(v[i].y, 1) : kept(v[i].z, 2));
                    if (mk) mk[e + j] = static_cast<u8>((m >> (8 * j)) & 1u);
                }
            }
        }
    }
#pragma unroll
    for (u32 g = 0; g < kMine; ++g) {
        const u32 b = b0 + g * kStripThreads;
        if (b >= n_blocks) continue;
        const u64 u = u0 + b;
        a.keys[u] = key[g];
        if (sumsq) sumsq[u] = acc[g];
        if (norms) norms[u] = static_cast<float>(sqrt(acc[g]));
        if (place[g] < room) {
            const u64 to = (static_cast<u64>(list_at[g]) << s.log_room) + place[g];
            s.key[to] = key[g];
            s.id[to] = static_cast<u32>(u);
        }
    }
}

// ---- after the sweep ---------------------------------------------------------------------------------------

struct StripFound {        // the threshold
    u64 T;
    u32 rem, n_tie;        // of its equals, how many are kept and how many there are
    u64 tie_end;
};

struct StripShared {
    u64 key[kStripMostSlots];
    u32 id[kStripMostSlots];
    u32 cnt[kStripPassBins];
    u64 most[kStripPassBins], leastc[kStripPassBins];
    uint2 queue[kStripSettle];          // blocks decided wrongly: id, tensor << 1 | kept
    u64 T, tie_end, a, b;
    u32 wave[kResolveThreads / 64];
    u32 rem, n_tie, n, bin, rank, found, over, n_queue[3];
};

// Writes the listed blocks again, a quad or an element (of s.units to a block) at a time: a workgroup has a few of them as a rule, but all of its
// blocks may be equal and decided by their place.
__device__ inline void strip_rewrite(const StructArgs& a, const StripArgs& s, const StripShared& sh, u32 n) {
    const u32 items = n * s.units;
    constexpr u32 kAtOnce = 2;
    for (u32 i0 = threadIdx.x; i0 < items; i0 += kAtOnce * kResolveThreads) {
        u64 e[kAtOnce];
        float* theta[kAtOnce];
        u8* mask[kAtOnce];
        float4 x[kAtOnce];
        bool keep[kAtOnce], there[kAtOnce];
#pragma unroll
        for (u32 j = 0; j < kAtOnce; ++j) {
            const u32 i = i0 + j * kResolveThreads, q = fast_div(i < items ? i : 0u, s.by_units), c = (i < items ? i : 0u) - q * s.units;
            const uint2 entry = sh.queue[q];
            const int t = static_cast<int>(entry.y >> 1);
            const TensorDesc& td = a.td[t];
            const u32 d2 = td.d[2], d3 = td.d[3], b2 = td.b[2], b3 = td.b[3];
            const u32 G3 = fast_div(d3 + b3 - 1, td.fd[kDivB3]), b = entry.x - static_cast<u32>(td.struct_start), g2 = b / G3, g3 = b - g2 * G3;
            const u32 h = d2 - g2 * b2 < b2 ? d2 - g2 * b2 : b2, wd = d3 - g3 * b3 < b3 ? d3 - g3 * b3 : b3;
            const u32 per = s.quad ? 4u : 1u, in_row = wd / per, row = ((((1u << 20) + in_row - 1) / in_row) * c) >> 20;         // c < 256
            keep[j] = (entry.y & 1u) != 0;
            there[j] = i < items && row < h;
            e[j] = (static_cast<u64>(g2) * b2 + (there[j] ? row : 0u)) * d3 + static_cast<u64>(g3) * b3 + (there[j] ? (c - row * in_row) * per : 0u);
            theta[j] = s.out[t].theta;
            mask[j] = s.out[t].mask;
            x[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (keep[j] && there[j]) { if (s.quad) x[j] = *reinterpret_cast<const float4*>(td.w + e[j]); else x[j].x = td.w[e[j]]; }
        }
#pragma unroll
        for (u32 j = 0; j < kAtOnce; ++j) {
            if (!there[j]) continue;
            if (s.quad) {
                if (theta[j]) *reinterpret_cast<float4*>(theta[j] + e[j]) = x[j];
                if (mask[j]) *reinterpret_cast<u32*>(mask[j] + e[j]) = keep[j] ? 0x01010101u : 0u;
            } else {
                if (theta[j]) theta[j][e[j]] = x[j].x;
                if (mask[j]) mask[j][e[j]] = keep[j] ? 1 : 0;
            }
        }
    }
}

__device__ inline void strip_keys(const StructArgs& a, u64 i0, u64 (&key)[kMaskPer]) {       // of four neighbours; those that there are not read 0
    if (i0 + kMaskPer <= a.F) {
        const ulonglong2 x = *reinterpret_cast<const ulonglong2*>(a.keys + i0), y = *reinterpret_cast<const ulonglong2*>(a.keys + i0 + 2);
        key[0] = x.x; key[1] = x.y; key[2] = y.x; key[3] = y.y;
    } else {
#pragma unroll
        for (int k = 0; k < kMaskPer; ++k) key[k] = i0 + k < a.F ? a.keys[i0 + k] : 0;
    }
}
// The tensor of block u, the same for all lanes of a wavefront.
__device__ inline int strip_tensor_of(const StructArgs& a, u64 u) {
    const u32 lane = threadIdx.x & 63u, n = static_cast<u32>(a.n_tensors);
    u32 upto = 0;
    for (u32 t0 = 0; t0 < n; t0 += 64) upto += static_cast<u32>(__popcll(__ballot(t0 + lane < n && a.td[t0 + lane < n ? t0 + lane : 0].struct_start <= u)));
    return static_cast<int>(upto) - 1;
}
// Structure mask, kept ids and corrections of blocks id0 .. id1 - 1, of whose predecessors `before` are kept.  `key`: strip_keys of this thread's first blocks, from id0 rounded down to a multiple of four; t0: id0's tensor.
template <bool REWRITE>
__device__ inline void strip_settle(const StructArgs& a, const StripArgs& s, StripShared& sh, const StripFound& f, u32 mid, u64 id0, u64 id1, u32 before, int t0,
                                    u64 (&key)[kMaskPer]) {
    const u32 tid = threadIdx.x;
    if (id0 >= id1) return;                                // uniform
    const u64 next_start = a.td[t0 + 1].struct_start;
    const bool wide = (reinterpret_cast<uintptr_t>(s.user_mask) & 3u) == 0;
    if (REWRITE && tid < 3) sh.n_queue[tid] = 0;
    __syncthreads();
    u32 turn = 0;                                          // whose queue it is: the one after it is cleared when all have left the one before it
    for (u64 base = id0 & ~static_cast<u64>(kMaskPer - 1); base < id1; base += kStripSettle) {
        const u64 i0 = base + tid * kMaskPer;
        const bool full = i0 >= id0 && i0 + kMaskPer <= id1;
        u64 next[kMaskPer] = {0, 0, 0, 0};
        if (base + kStripSettle < id1) strip_keys(a, i0 + kStripSettle, next);         // on their way
        const u32 after = turn == 2 ? 0u : turn + 1;
        if (REWRITE && tid == 0 && base + kStripSettle < id1) sh.n_queue[after] = 0;
        u32 keep[kMaskPer], n = 0;
#pragma unroll
        for (int k = 0; k < kMaskPer; ++k) {
            const u64 u = i0 + k;
            const bool there = u >= id0 && u < id1;
            keep[k] = there && (key[k] > f.T || (key[k] == f.T && u < f.tie_end)) ? 1u : 0u;
            n += keep[k];
            const u32 was = static_cast<u32>(key[k] >> 32) >= mid ? 1u : 0u;
            if (REWRITE && there && was != keep[k]) {
                int t = t0;
                if (u >= next_start) while (t + 1 < a.n_tensors && a.td[t + 1].struct_start <= u) ++t;
                sh.queue[atomicAdd(&sh.n_queue[turn], 1u)] = make_uint2(static_cast<u32>(u), static_cast<u32>(t) << 1 | keep[k]);
            }
        }
        if (s.user_mask) {
            if (full && wide) {
                *reinterpret_cast<uchar4*>(s.user_mask + i0) = make_uchar4(static_cast<u8>(keep[0]), static_cast<u8>(keep[1]), static_cast<u8>(keep[2]), static_cast<u8>(keep[3]));
            } else {
#pragma unroll
                for (int k = 0; k < kMaskPer; ++k) if (i0 + k >= id0 && i0 + k < id1) s.user_mask[i0 + k] = static_cast<u8>(keep[k]);
            }
        }
        u32 total;
        u32 pos = before + wg_incl_scan_u32<kResolveThreads>(n, sh.wave, &total) - n;    // (a barrier: the queue is complete)
        before += total;
        if (s.keep_idx) {
#pragma unroll
            for (int k = 0; k < kMaskPer; ++k) if (keep[k] && pos < a.F) s.keep_idx[pos++] = static_cast<int32_t>(i0 + k);
        }
#pragma unroll
        for (int k = 0; k < kMaskPer; ++k) key[k] = next[k];
        if (!REWRITE) continue;
        const u32 n_queue = sh.n_queue[turn];
        turn = after;
        if (n_queue == 0) continue;                        // uniform
        strip_rewrite(a, s, sh, n_queue);
        __syncthreads();                                   // the queue is used again
    }
}

__device__ inline void strip_record(const StructArgs& a, const StripArgs& s, const StripFound& f) {
    const Slot& slot = a.slots[0];
    condensa_select out;
    out.n = slot.n;
    out.k = slot.k;
    out.n_gt = slot.k - f.rem;
    out.n_tie_kept = f.rem;
    out.n_tie = f.n_tie;
    out.threshold_key = f.T;
    out.tie_end = f.tie_end;
    out.path = slot.path;
    *s.results = out;
}

// The last block kept of n in LDS, the want-th from the top.
__device__ inline StripFound strip_rank(StripShared& sh, u32 n, u32 want, u64 n_all) {
    const u32 tid = threadIdx.x;
    for (u32 i0 = 0; i0 < n; i0 += kResolveThreads / 4) {  // four threads to an entry
        const u32 i = i0 + tid / 4;
        const u64 key = sh.key[i < n ? i : 0];
        const u32 id = sh.id[i < n ? i : 0];
        u32 higher = 0, same = 0, lower = 0;
        for (u32 e = tid % 4; e < n; e += 4) {
            const u64 o = sh.key[e];
            higher += o > key ? 1u : 0u;
            same += o == key ? 1u : 0u;
            lower += o == key && sh.id[e] < id ? 1u : 0u;
        }
#pragma unroll
        for (int d = 1; d < 4; d *= 2) {
            higher += __shfl_xor(higher, d, 64);
            same += __shfl_xor(same, d, 64);
            lower += __shfl_xor(lower, d, 64);
        }
        if (i < n && tid % 4 == 0 && higher < want && want <= higher + same && lower == want - higher - 1) {       // the last one kept: one thread
            sh.T = key;
            sh.rem = want - higher;
            sh.n_tie = same;
            sh.tie_end = want - higher == same ? n_all : static_cast<u64>(id) + 1;
        }
    }
    __syncthreads();
    return StripFound{sh.T, sh.rem, sh.n_tie, sh.tie_end};
}

// What the places of the bins do not tell: all workgroups that are running, over all keys.  A pass counts the keys of an interval in
// kStripPassBins bins and keeps every bin's greatest and least key, so a bin of equal keys ends the search.  One of few keys too: they are gathered, and everybody
// ranks them (2^20 blocks of 4x4 in two scales, the threshold at the gap between them: two
// passes and two meetings less, and the counters of the bins are not looked at where none were filled: the call 92.3 -> 82.4 us).
__device__ inline void strip_fallback(const StructArgs& a, const StripArgs& s, StripShared& sh, const ListWin& win) {
    const u32 tid = threadIdx.x;
    Meet m;
    if (!meet_join(m, s.meet, sh.wave)) return;
    const u64 i0 = a.F * m.rank / m.size, i1 = a.F * (m.rank + 1) / m.size, k = a.slots[0].k;
    u64 lo = static_cast<u64>(win.lo) << 32, hi = (static_cast<u64>(win.hi) << 32) | 0xFFFFFFFFull, rank = 0;          // rank 0: the interval is a guess
    u32 tie_here = 0, above_here = 0, kept_before = 0;     // kept_before: of the blocks before this workgroup's share
    bool gathered = false;
    StripFound f{0, 0, 0, 0};
    auto share = [&](auto&& g) {                           // g(block, key) for this workgroup's, several loads at a time
        constexpr int kAtOnce = 8;
        for (u64 base = i0; base < i1; base += kAtOnce * kResolveThreads) {
            u64 there[kAtOnce];
#pragma unroll
            for (int j = 0; j < kAtOnce; ++j) { const u64 i = base + j * kResolveThreads + tid; there[j] = a.keys[i < i1 ? i : base]; }
#pragma unroll
            for (int j = 0; j < kAtOnce; ++j) { const u64 i = base + j * kResolveThreads + tid; if (i < i1) g(i, there[j]); }
        }
    };
    for (u32 pass = 0;; ++pass) {                          // uniform over all workgroups; at most eight
        if (pass == 32) return;
        u32* const set = s.pass + pass % 3 * kStripPassWords;
        u32* const g_cnt = set;
        u64* const g_most = reinterpret_cast<u64*>(set + kStripPassBins);
        u64* const g_leastc = g_most + kStripPassBins;
        u32* const g_above = set + 5 * kStripPassBins;
        const u64 span = hi - lo;
        const u32 shift = span < kStripPassBins ? 0u : static_cast<u32>(64 - kStripPassBits - __clzll(static_cast<long long>(span)));
        static_assert(kStripPassBins == 2 * kResolveThreads, "two bins a thread");
        for (u32 i = tid; i < kStripPassBins; i += kResolveThreads) { sh.cnt[i] = 0; sh.most[i] = 0; sh.leastc[i] = 0; }
        __syncthreads();
        u32 above = 0;
        share([&](u64, u64 key) {
            if (key > hi) ++above;
            else if (key >= lo) {
                const u32 bin = static_cast<u32>((key - lo) >> shift);
                atomicAdd(&sh.cnt[bin], 1u);
                atomicMax(reinterpret_cast<unsigned long long*>(&sh.most[bin]), static_cast<unsigned long long>(key));
                atomicMax(reinterpret_cast<unsigned long long*>(&sh.leastc[bin]), static_cast<unsigned long long>(~key));
            }
        });
        u32 above_all;
        wg_incl_scan_u32<kResolveThreads>(above, sh.wave, &above_all);
        for (u32 i = tid; i < kStripPassBins; i += kResolveThreads) {
            if (sh.cnt[i] == 0) continue;
            add_dev(g_cnt + i, sh.cnt[i]);
            __hip_atomic_fetch_max(g_most + i, sh.most[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_max(g_leastc + i, sh.leastc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (tid == 0 && above_all) add_dev(g_above, above_all);
        // the next pass's set: all have left the pass that used it, the one before the last
        u32* const clear = s.pass + (pass + 1) % 3 * kStripPassWords;
        if (pass > 1) for (u32 i = m.rank * kResolveThreads + tid; i < kStripPassWords; i += m.size * kResolveThreads) st_dev(clear + i, 0u);
        meet(m);
        // bins from the top, two a thread
        const u32 top = kStripPassBins - 1 - 2 * tid;
        const u32 c0 = ld_dev(g_cnt + top), c1 = ld_dev(g_cnt + top - 1);
        u32 inside;
        const u32 upto = wg_incl_scan_u32<kResolveThreads>(c0 + c1, sh.wave, &inside);
        if (rank == 0) {                                   // uniform, the first pass: does the interval hold the threshold?
            const u64 beyond = ld_dev(g_above);
            if (beyond >= k) { lo = hi + 1; hi = 0x7FFFFFFFFFFFFFFFull; rank = k; continue; }
            if (k - beyond > inside) { hi = lo - 1; lo = 0; rank = k - beyond - inside; continue; }
            rank = k - beyond;
        }
        const u32 before = upto - c0 - c1, r = static_cast<u32>(rank);
        if (before < r && r <= upto) {                     // one thread
            const bool first = r <= before + c0;
            sh.bin = first ? top : top - 1;
            sh.rank = first ? r - before : r - before - c0;
            sh.n = first ? c0 : c1;
            sh.a = ~ld_dev64(g_leastc + sh.bin);
            sh.b = ld_dev64(g_most + sh.bin);
        }
        __syncthreads();
        lo = sh.a; hi = sh.b; rank = sh.rank;
        const bool done = lo == hi;
        gathered = !done && sh.n <= kStripGather;
        if (done || gathered) {
            f.T = lo; f.rem = static_cast<u32>(rank); f.n_tie = sh.n;
            u32 higher = 0;                                // this share's, in the bins above
            for (u32 i = tid; i < kStripPassBins; i += kResolveThreads) if (i > sh.bin) higher += sh.cnt[i];
            wg_incl_scan_u32<kResolveThreads>(higher, sh.wave, &above_here);
            above_here += above_all;
            tie_here = sh.cnt[sh.bin];
        }
        __syncthreads();
        if (gathered) {                                    // the next pass's set is cleared; one of its spare words counts
            u32* const n_there = s.pass + (pass + 1) % 3 * kStripPassWords + 5 * kStripPassBins + 1;
            if (tid == 0) {
                st_dev(s.share + m.rank, above_here);
                sh.n_queue[0] = tie_here ? add_dev(n_there, tie_here) : 0u;
            }
            __syncthreads();
            if (tie_here) share([&](u64 i, u64 key) {
                if (key < lo || key > hi) return;
                const u32 to = atomicAdd(&sh.n_queue[0], 1u);            // f.n_tie of them
                st_dev64(s.key + to, key);
                st_dev(s.id + to, static_cast<u32>(i));
            });
            meet(m);
            for (u32 i = tid; i < f.n_tie; i += kResolveThreads) { sh.key[i] = ld_dev64(s.key + i); sh.id[i] = ld_dev(s.id + i); }
            u32 before = 0;
            for (u32 i = tid; i < m.rank; i += kResolveThreads) before += ld_dev(s.share + i);
            __syncthreads();
            const u32 n = f.n_tie;
            f = strip_rank(sh, n, f.rem, a.slots[0].n);
            for (u32 i = tid; i < n; i += kResolveThreads) before += sh.id[i] < i0 && (sh.key[i] > f.T || (sh.key[i] == f.T && sh.id[i] < f.tie_end)) ? 1u : 0u;
            wg_incl_scan_u32<kResolveThreads>(before, sh.wave, &kept_before);
            break;
        }
        if (done) break;
    }
    if (!gathered) {
        if (tid == 0) {
            st_dev(s.share + m.rank, above_here);
            st_dev(s.share + kStripResolveGrid + m.rank, tie_here);
        }
        meet(m);
        u32 above = 0, ties = 0, above_before, ties_before;
        for (u32 i = tid; i < m.rank; i += kResolveThreads) { above += ld_dev(s.share + i); ties += ld_dev(s.share + kStripResolveGrid + i); }
        wg_incl_scan_u32<kResolveThreads>(above, sh.wave, &above_before);
        wg_incl_scan_u32<kResolveThreads>(ties, sh.wave, &ties_before);
        f.tie_end = a.slots[0].n;
        if (f.rem < f.n_tie) {                                 // the last tie kept is in one of the shares
            if (ties_before < f.rem && f.rem <= ties_before + tie_here) {
                u32 seen = ties_before;
                for (u64 base = i0; base < i1; base += kResolveThreads) {
                    const u64 i = base + tid;
                    const u32 eq = i < i1 && a.keys[i] == f.T ? 1u : 0u;
                    u32 total;
                    const u32 upto = seen + wg_incl_scan_u32<kResolveThreads>(eq, sh.wave, &total);
                    if (eq && upto == f.rem) st_dev64(s.tie_end, i + 1);
                    seen += total;
                    if (seen >= f.rem) break;                  // uniform
                }
            }
            meet(m);
            f.tie_end = ld_dev64(s.tie_end);
        }
        kept_before = above_before + (ties_before < f.rem ? ties_before : f.rem);
    }
    if (m.rank == 0 && tid == 0) strip_record(a, s, f);
    // The blocks decided wrongly may be neighbours (equal ones up to the last tie kept), so everybody takes a few of everywhere.
    const u32 mid = strip_mid(win);
    const u64 stride = static_cast<u64>(m.size) * kResolveThreads;
    for (u64 base = static_cast<u64>(m.rank) * kResolveThreads; base < a.F; base += kMaskPer * stride) {
        u64 there[kMaskPer];
#pragma unroll
        for (int j = 0; j < kMaskPer; ++j) { const u64 u = base + j * stride + tid; there[j] = u < a.F ? a.keys[u] : 0; }
        if (tid == 0) sh.n_queue[0] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kMaskPer; ++j) {
            const u64 first = base + j * stride, u = first + tid;
            if (first >= a.F) break;                       // uniform
            const u32 keep = there[j] > f.T || (there[j] == f.T && u < f.tie_end) ? 1u : 0u, was = static_cast<u32>(there[j] >> 32) >= mid ? 1u : 0u;
            int t = strip_tensor_of(a, first);
            if (u < a.F && keep != was) {
                while (t + 1 < a.n_tensors && a.td[t + 1].struct_start <= u) ++t;
                sh.queue[atomicAdd(&sh.n_queue[0], 1u)] = make_uint2(static_cast<u32>(u), static_cast<u32>(t) << 1 | keep);
            }
        }
        __syncthreads();
        const u32 n = sh.n_queue[0];
        if (n) strip_rewrite(a, s, sh, n);                 // uniform
        __syncthreads();                                   // the queue is used again
    }
    if (i0 >= i1) return;                                  // uniform
    u64 key[kMaskPer];
    strip_keys(a, (i0 & ~static_cast<u64>(kMaskPer - 1)) + tid * kMaskPer, key);
    strip_settle<false>(a, s, sh, f, mid, i0, i1, kept_before, strip_tensor_of(a, i0), key);
}

// Bound by latency: a launch and a chain of some six dependent loads -- the counters, the counters of one thread's bins, the places of the bins
// in question, a wrong block's descriptor and weights; what does not depend on them is on its way meanwhile.
__global__ __launch_bounds__(kResolveThreads) void k_strip_resolve(StructArgs a, StripArgs s) {
    __shared__ StripShared sh;
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 t0 = static_cast<u32>(static_cast<u64>(s.n_tiles) * blockIdx.x / gridDim.x), t1 = static_cast<u32>(static_cast<u64>(s.n_tiles) * (blockIdx.x + 1) / gridDim.x);
    const u64 id0 = s.tiles[t0].x, id1 = s.tiles[t1].x;
    const ListWin win = *s.win;
    if (!strip_listed(win)) {                              // uniform, the same in every workgroup
        strip_fallback(a, s, sh, win);
        return;
    }
    const u32 bins = 1u << s.log_bins, shift = strip_shift(win, s.log_bins), k = static_cast<u32>(a.slots[0].k), mid = strip_mid(win);
    // what comes before this workgroup's strips, and what lies above the window
    u32 above = tid < kStripAboves ? s.above[tid * kListLine] : 0u, before = 0;
    if (s.keep_idx) {
        for (u32 i = tid; i < t0 >> s.log_group; i += kResolveThreads) before += s.coarse[i * kListLine];
        for (u32 i = (t0 >> s.log_group << s.log_group) + tid; i < t0; i += kResolveThreads) before += s.tiles[i].y;
    }
    // (counting the blocks by runs of bins too, so that 32 KB need not be read, cost the sweep 3 us and gained 1)
    const uint4* const counts = reinterpret_cast<const uint4*>(s.hist);      // of a bin
    static_assert(kStripCopies == 4, "a bin's counters are loaded together");
    const u32 per = bins > static_cast<u32>(kResolveThreads) ? bins / kResolveThreads : 1u;           // bins of a thread, from the top
    u32 sum = 0;
    for (u32 i = 0; i < per; i += 4) {
        uint4 c[4];
#pragma unroll
        for (u32 j = 0; j < 4; ++j) c[j] = counts[bins - 1 - (tid * per + i + j < bins ? tid * per + (i + j < per ? i + j : i) : 0u)];
#pragma unroll
        for (u32 j = 0; j < 4; ++j) sum += i + j < per && tid * per + i + j < bins ? c[j].x + c[j].y + c[j].z + c[j].w : 0u;
    }
    u64 mine[kMaskPer];                                    // the keys that this thread settles first
    strip_keys(a, (id0 & ~static_cast<u64>(kMaskPer - 1)) + tid * kMaskPer, mine);
    const int tensor = strip_tensor_of(a, id0);
    if (tid == 0) { sh.found = 0; sh.over = 0; sh.n = 0; }
    u32 inside;
    wg_incl_scan_u32<kResolveThreads>(above, sh.wave, &above);
    const u32 upto = wg_incl_scan_u32<kResolveThreads>(sum, sh.wave, &inside);
    const u32 r = k - above;                               // wanted among the listed ones, if 1 <= r <= inside
    if (above < k && upto - sum < r && r <= upto) { sh.a = tid; sh.rank = r - (upto - sum); sh.found = 1; }      // one thread at most
    __syncthreads();
    if (sh.found && tid < 64) {                            // its bins, a lane each
        const u32 bin = bins - 1 - (static_cast<u32>(sh.a) * per + lane), want = sh.rank;
        static_assert(kStripMostBins / kResolveThreads <= 64, "a lane a bin");
        const uint4 c = lane < per ? counts[bin] : make_uint4(0, 0, 0, 0);
        const u32 n = c.x + c.y + c.z + c.w, incl = wave_incl_scan_u32(n);
        if (incl - n < want && want <= incl) { sh.bin = bin; sh.rank = want - (incl - n); }
    }
    __syncthreads();
    const bool found = sh.found != 0;
    const u32 bin = sh.bin, want = sh.rank, mid_bin = (win.mid - win.lo) >> shift;
    // The places of the bins between the estimate and the threshold, which lies in one of them; one that has no room for its blocks leaves it to the fallback.  Of the blocks
    // there that come before this workgroup's, those in other bins than the threshold's were decided wrongly.
    const u32 first = bin < mid_bin ? bin : mid_bin, last = bin < mid_bin ? mid_bin - 1 : bin;
    const u32 n_places = found ? (last - first + 1) * kStripCopies : 0u;
    u32 over = 0, wrong = 0;
    const u32 room = 1u << s.log_room, slots = kStripCopies << s.log_room;
    for (u32 i = tid; found && i < slots; i += kResolveThreads) {        // the threshold's
        const u32 at = bin * slots + i, have = s.hist[at >> s.log_room], id = s.id[at];                  // (garbage where there is no block)
        const u64 key = s.key[at];
        over |= have > room ? 1u : 0u;
        if ((at & (room - 1)) < have) {
            const u32 to = atomicAdd(&sh.n, 1u);
            sh.key[to] = key;
            sh.id[to] = id;
        }
    }
    // A thread looks at the blocks of one copy of a bin, some ten: at eight at once without waiting for their number.
    for (u32 i0 = tid; i0 < n_places; i0 += 2 * kResolveThreads) {
        u32 have[2];
        uint4 id[2][2];
#pragma unroll
        for (u32 j = 0; j < 2; ++j) {
            const u32 i = i0 + j * kResolveThreads, at = first * kStripCopies + (i < n_places ? i : i0);
            have[j] = s.hist[at];
            id[j][0] = *reinterpret_cast<const uint4*>(s.id + (at << s.log_room));
            id[j][1] = *reinterpret_cast<const uint4*>(s.id + (at << s.log_room) + 4);
        }
#pragma unroll
        for (u32 j = 0; j < 2; ++j) {
            const u32 i = i0 + j * kResolveThreads, at = first * kStripCopies + i;
            if (i >= n_places || at / kStripCopies == bin) continue;
            over |= have[j] > room ? 1u : 0u;
            auto count = [&](const uint4& x, u32 from) {
                wrong += (from < have[j] && x.x < id0 ? 1u : 0u) + (from + 1 < have[j] && x.y < id0 ? 1u : 0u) +
                         (from + 2 < have[j] && x.z < id0 ? 1u : 0u) + (from + 3 < have[j] && x.w < id0 ? 1u : 0u);
            };
            count(id[j][0], 0);
            count(id[j][1], 4);
            const uint4* const more = reinterpret_cast<const uint4*>(s.id + (at << s.log_room));
            for (u32 from = 8; from < room && from < have[j]; from += 8) {
                const uint4 x = more[from / 4], y = more[from / 4 + 1];
                count(x, from);
                count(y, from + 4);
            }
        }
    }
    if (over) sh.over = 1;
    __syncthreads();
    if (!found || sh.over) {                               // uniform, and the same in every workgroup
        __syncthreads();
        strip_fallback(a, s, sh, win);
        return;
    }
    const u32 n = sh.n;
    const StripFound f = strip_rank(sh, n, want, a.slots[0].n);
    if (s.keep_idx) {
        // bins below the estimate's that turn out to be kept, bins from it on that do not, and the threshold's own
        u32 add = bin < mid_bin ? wrong : 0u - wrong;
        for (u32 i = tid; i < n; i += kResolveThreads) {
            if (sh.id[i] >= id0) continue;
            const bool keep = sh.key[i] > f.T || (sh.key[i] == f.T && sh.id[i] < f.tie_end), was = bin >= mid_bin;
            add += static_cast<u32>(keep) - static_cast<u32>(was);
        }
        u32 total;
        wg_incl_scan_u32<kResolveThreads>(before + add, sh.wave, &total);              // modulo 2^32: the sum is not negative
        before = total;
    }
    if (blockIdx.x == 0 && tid == 0) strip_record(a, s, f);
    strip_settle<true>(a, s, sh, f, mid, id0, id1, before, tensor, mine);
}

}  // namespace condensa
