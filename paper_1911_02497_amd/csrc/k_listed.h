// Listed windows: the selection of ordinary calls (the rule is want_list, either scope) in three to seven launches.
//
// Up to some ten million weights a call is bound by its dependent launches (about 4.5 us each, however little they
// do) and by how often it reads the weights, which the three histogram sweeps of the radix levels make four times.
// Here
//   1. k_list_sample: every workgroup ranks its own sample in LDS.  For a ranking it wants the sample keys at the
//      expected rank of the threshold and a little to either side of it.  Small populations get one workgroup, whose
//      bounds lie as many standard deviations of the sample rank apart as the call asks for.  Large ones get up to
//      kListMaxW, each with a sample spread over the whole population, and k_list_bounds takes order statistics of
//      their keys: a confidence interval for the threshold that needs no assumption about how neighbours correlate.
//      Either way: a window [lo, hi] that holds the threshold unless the sample was unlucky, and an estimate `mid`.
//   2. k_list_sweep / k_list_sweep_multi: ONE pass over the weights writes the outputs (final outside the windows,
//      provisional -- kept from `mid` on -- inside), counts the keys from `mid` on and lists the keys inside each
//      window with their indices.
//   3. k_list_hist counts each list in kListBins bins over its window; k_list_gather finds the bin of rank k - above,
//      settles the listed elements outside it (their outputs are rewritten where the provisional decision was wrong)
//      and gathers those inside, a few hundred.
//   4. k_list_settle ranks these, applies the tie rule, writes state and record and settles them too.  If some ranking
//      failed (its rank is not inside the window, or a list overflowed) it ranks that population by radix levels over
//      the weights instead and applies every result again.
// One workgroup draws some 25 GB/s from memory it did not write, so the lists (10^5 entries) are walked by many.  When
// no population exceeds list_lone elements, its list is short enough for one workgroup to do 3 and 4 alone
// (k_list_finish): three launches, and a failed ranking stays within that workgroup.
// Results never depend on the sample.  Section 3.1 (a sparsity turned into a magnitude threshold), Section 3.3 (the
// C step and the multiplier update), Results (up to ten samples per search share a pass).
#pragma once
#include "k_apply.h"
#include "k_small.h"
#include "k_window.h"

namespace condensa {

constexpr int kListThreads = 1024;
constexpr int kListUnits = 4;                    // sample positions (of four keys each) per thread of a lone workgroup; one of several takes one
constexpr int kListSegs = 1024;                  // segments of a ranking's list at most
constexpr int kListMaxW = 256;                   // sampling workgroups of one population at most
constexpr int kListMaxRankings = 4096;
constexpr int kListBins = 256;                   // bins over a window
constexpr u32 kListRanked = 2048;                // gathered entries that are held in LDS
constexpr u32 kListGather = 1u << 18;            // gathered entries of a ranking at most; with more (ties) it fails
constexpr u32 kListRow = 64;                     // segments are multiples of this many entries

// Populations up to here are finished by one workgroup.  Several densities: the windows of one sampling workgroup overlap,
// and the sweep's general path is slow.
__host__ __device__ inline u64 list_lone(int J) { return static_cast<u64>(1) << (J > 1 ? 16 : 18); }

// Sampling workgroups of a population of n elements: the window is narrowed as the population grows.  One workgroup leaves
// a window of up to 8 % of it (10 sd of its rank); 32 about 2 %, 64 about 1 %, 256 about 0.4 % at the cost of one more
// launch (4 us).  Above list_lone that launch is earned back at once: 295 thousand weights in two densities 52.3 us with one,
// 37.7 with 32; 600 thousand 59.7 and 39.5; pruning 700 thousand in one density 37.3 and 36.5.
__host__ __device__ inline u32 list_sample_groups(u64 n, int J) {
    if (n <= list_lone(J)) return 1;
    if (n <= (static_cast<u64>(1) << 21)) return 32;
    if (n <= (static_cast<u64>(1) << 23)) return 64;
    return kListMaxW;
}
// Entries of a ranking's list: several times what its window is expected to hold, every element of a tiny one.
inline u64 list_capacity(u64 n, int cand_shift) {
    if (cand_shift > 0) return (n >> cand_shift) < 4096 ? 4096 : n >> cand_shift;
    if (n <= 4096) return n;
    u64 c = n <= (static_cast<u64>(1) << 21) ? n / 4 : n / 16;
    const u64 least = n <= (static_cast<u64>(1) << 21) ? 4096 : (static_cast<u64>(1) << 19);
    return c < least ? least : c;
}
// Segments of a list that wavefronts of `per_wave` elements append to: updates of one counter that return a value
// take turns (some 0.15 us each under contention), so a counter serves four wavefronts while segments last.  Always an
// odd number: a workgroup takes the segment of its number, and tensors that leave the same part of every chunk empty
// would otherwise leave the same segments empty.
inline u32 list_segments(u64 n, u64 per_wave, u32 most) {
    const u64 s = n / (4 * per_wave);
    return s < 1 ? 1u : ((s >= most ? most - 1 : static_cast<u32>(s)) | 1u);
}

// Window of a ranking.  Its keys fall into bins (key - lo) >> shift; the estimate `mid` is the lower edge of bin mid_bin.
// lo = hi = mid = 2^32 - 1: nothing is kept, nothing listed.
struct ListWin { u32 lo, hi, mid, bins; };       // bins: shift | mid_bin << 8

// Several rankings of one population: their windows in descending order, for k_list_sweep_multi.  A key's region is the
// number of estimates `mid` that it reaches; while no two windows overlap it tells every decision, and the key can only be
// inside the window of the highest estimate it reaches or of the next one up.
struct ListSorted {
    u32 mid[kMaxJ];        // descending; n of them (rankings with nothing to select are left out)
    u32 gap_lo[kMaxJ + 1]; // region r: keys outside every window are gap_lo .. gap_lo + gap_len - 1
    u32 gap_len[kMaxJ + 1];
    u32 ranking[kMaxJ];    // at each position
    u32 bias[kMaxJ];       // by ranking: 127 - c, where the region must exceed c for the key to be kept
    u32 n;
    u32 disjoint;
    u32 unused[2];
};

struct ListRank {          // one ranking: filled by the host
    u64 base;              // its first list entry
    u32 seg_cap;           // entries per segment, a multiple of kListRow
    u32 n_segs;
    u32 group0;            // first sampling workgroup of its population
    u32 n_groups;          // how many
    u32 unused[2];
};
static_assert(sizeof(ListRank) == 32, "ListRank layout");

struct FallbackCtl {       // cleared at the start of every call
    u32 failed;            // rankings that the window path did not resolve
    u32 ticket;
    u32 done;
    u32 unused;
};

struct ListArgs {
    const ListRank* rank;  // [rankings]
    const u32* group_of;   // PER_TENSOR: [sampling workgroups] tensor each samples
    ListWin* local;        // [sampling workgroups][J]
    ListWin* win;          // [rankings]
    ListSorted* sorted;    // [populations], J > 1
    u64* cnt;              // [rankings][max_segs] entries offered | keys at or above `mid` << 32
    u32* hist;             // [rankings][kListBins]
    u32* gathered;         // [rankings] entries in the threshold's bin
    u32* bin_want;         // [rankings] rank to find among them
    u32* gkey;             // [rankings][gather_cap]
    u32* gidx;
    u32 gather_cap;
    u32 parts;             // workgroups per ranking that walk a list
    u32* nnz;              // [kListSegs] prune + binary16 step: provisional non-zero codes
    u32 max_segs;          // counters per ranking
    int n_rankings;
    u32* key;
    u32* idx;              // element as chunk * kChunk + place in the chunk: the order of flat indices, and the
                           // tensor is one look-up away
    FallbackCtl* fb;
    u32* fail_list;        // [rankings]
    u32* fb_hist;          // [2][3][kBins]
    const OutDesc* out;
    u64* nnz_out;
    int margin16;
    int write;             // 1: the sweep writes the outputs.  0: selection only, an apply sweep follows
};

// ---- sample ------------------------------------------------------------------------------------------

__device__ inline ListWin list_window(u32 hi, u32 lo, u32 mid) {
    ListWin x;
    x.hi = hi;
    x.lo = hi == 0xFFFFFFFFu ? hi : (lo < hi ? lo : hi);
    mid = mid < x.lo ? x.lo : (mid > x.hi ? x.hi : mid);
    u32 shift = 0;
    while (((x.hi - x.lo) >> shift) >= static_cast<u32>(kListBins)) ++shift;
    const u32 mid_bin = (mid - x.lo) >> shift;
    x.mid = x.lo + (mid_bin << shift);
    x.bins = shift | (mid_bin << 8);
    return x;
}

// One wavefront, J <= kMaxJ windows (in LDS), `by_rank` kMaxJ + 1 words of LDS.  Lane j places window j.
__device__ inline void list_sort(const ListWin* win, int J, u32* by_rank, ListSorted* out) {
    const int lane = threadIdx.x & 63;
    const ListWin mine = lane < J ? win[lane] : ListWin{};
    const bool active = lane < J && mine.hi != 0xFFFFFFFFu;
    const u32 n = static_cast<u32>(__popcll(__ballot(active)));
    u32 p = 0;                                             // windows before this one: higher, or equal and earlier
    for (int i = 0; i < J; ++i) {
        const u32 h = win[i].hi;
        if (h != 0xFFFFFFFFu && (h > mine.hi || (h == mine.hi && i < lane))) ++p;
    }
    if (active) by_rank[p] = static_cast<u32>(lane);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const ListWin next = active && p + 1 < n ? win[by_rank[p + 1]] : ListWin{0, 0, 0, 0};
    const u64 overlap = __ballot(active && p + 1 < n && next.hi >= mine.lo);
    if (lane < J) out->bias[lane] = active ? 127u - (n - p - 1u) : 0u;   // nothing selected: no region reaches it
    if (active) {
        out->mid[p] = mine.mid;
        out->ranking[p] = static_cast<u32>(lane);
        // region n - p - 1 lies below this window and above the next one, if there is one
        const u32 from = p + 1 < n ? next.hi + 1u : 0u;
        out->gap_lo[n - p - 1] = from;
        out->gap_len[n - p - 1] = mine.lo - from;
        if (p == 0) { out->gap_lo[n] = mine.hi + 1u; out->gap_len[n] = 0xFFFFFFFFu - (mine.hi + 1u); }
    }
    if (lane == 0) {
        if (n == 0) { out->gap_lo[0] = 0; out->gap_len[0] = 0xFFFFFFFFu; }
        out->n = n;
        out->disjoint = overlap == 0 ? 1u : 0u;
    }
}

// The bin of 256 that holds descending rank r (1 <= r <= all counts together): one wavefront, four bins per lane from
// the top.  The lane that finds it returns true.
__device__ inline bool wave_pick256(const u32* s_hist, u32 r, u32* bin) {
    const u32 lane = threadIdx.x & 63u;
    const uint4 c = *reinterpret_cast<const uint4*>(s_hist + 252 - 4 * lane);
    u32 incl = c.x + c.y + c.z + c.w;
    const u32 sum = incl;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const u32 up = __shfl_up(incl, d, 64);
        if (static_cast<int>(lane) >= d) incl += up;
    }
    u32 before = incl - sum;
    if (!(before < r && r <= incl)) return false;
    u32 b = 255 - 4 * lane;
    before += c.w;
    if (r > before) { --b; before += c.z; if (r > before) { --b; before += c.y; if (r > before) --b; } }
    *bin = b;
    return true;
}

// Where a sampling workgroup finds things: the tensor of a chunk, and a ranking's k (0: nothing to select) and n.
struct SampleTensor {
    const float* w;
    const float* lam;
    u64 n, chunk_start;
};

// One sampling workgroup of a population: number `me` of W, whose results go to place `at_local`.  Bound by latency
// (scattered 16-byte reads, then a dozen barriers).  A lone workgroup writes the window: the rank rule is that of
// sample_rank.  One of several leaves the keys at its expected rank and two ranks to either side of it (which covers
// the bias of small ranks); k_list_bounds does the rest.  `first_chunk`, `quads`: the population in chunk space.
template <bool LC, bool VEC, typename TensorOf, typename RankOf>
__device__ inline void list_sample(const ListArgs& w, int J, float mu, u32 W, u32 me, u32 at_local, u64 first_ranking, u64 first_chunk, u64 quads,
                                   TensorOf&& tensor_of, RankOf&& rank_of) {
    constexpr int kBits2 = 8, kBins2 = 1 << kBits2;        // 19 of 31 bits: the rest is a twentieth of a percent of the value
    __shared__ __align__(16) u32 s_hist[3 * kMaxJ * kBins2];   // level 0: one or four copies of 2048 bins; level 1: 3 J x kBins2
    __shared__ u8 s_tab[kBins];                  // leading digit -> 1 + histogram of level 1
    __shared__ ListWin s_win[kMaxJ];
    __shared__ u32 s_wave[kListThreads / 64];
    __shared__ u32 s_want[3 * kMaxJ], s_bin[3 * kMaxJ], s_rem[3 * kMaxJ], s_key[3 * kMaxJ];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int R = 3 * J;
    // A lone workgroup reads single float4; one of several reads 64-byte lines, four lanes each: the same traffic for four
    // times the keys (262144 scattered float4 of two arrays took 11 us), and order statistics do not mind neighbours that
    // resemble each other.
    const int units = W == 1 ? kListUnits : 1, lanes = W == 1 ? 1 : 4;
    const int logu = 31 - __clz(static_cast<int>(units * (kListThreads / lanes) * W));     // a power of two
    const u64 places = (quads + lanes - 1) / lanes;

    u32 key[4 * kListUnits], valid = 0;
#pragma unroll
    for (int i = 0; i < kListUnits; ++i) {
        if (i >= units) break;                   // uniform
        const u64 u = static_cast<u64>(i * kListThreads + tid / lanes) * W + me;
        u64 p = places <= (static_cast<u64>(1) << logu) ? u : (u * places + __umul64hi(static_cast<u64>(mix32(static_cast<u32>(u))) << 32, places)) >> logu;
        p = p * lanes + tid % lanes;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if (p < quads) {
            const u64 c = first_chunk + p / (kChunk / 4);
            const SampleTensor td = tensor_of(c);
            const u64 e0 = (c - td.chunk_start) * kChunk + (p % (kChunk / 4)) * 4;
            if (e0 < td.n) {
                load4<VEC>(td.w, e0, td.n, v);
                if (LC) {
                    float l[4];
                    load4<VEC>(td.lam, e0, td.n, l);
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = lc_shift(v[k], l[k], mu);
                }
                const u32 have = td.n - e0 < 4 ? static_cast<u32>(td.n - e0) : 4u;
                valid |= ((1u << have) - 1u) << (4 * i);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) key[4 * i + k] = mag_key(v[k]);
    }
    constexpr int kShift0 = 20;                  // 11 leading bits of 31
    const int copies = units == 1 ? 1 : 4;       // chosen by lane: fewer lanes of a wavefront meet on one counter
    for (int i = tid; i < copies * kBins; i += kListThreads) s_hist[i] = 0;
    for (int i = tid; i < kBins; i += kListThreads) s_tab[i] = 0;
    if (tid < R) s_bin[tid] = 0xFFFFFFFFu;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4 * kListUnits; ++i)
        if (valid & (1u << i)) atomicAdd(&s_hist[(lane & (copies - 1)) * kBins + (key[i] >> kShift0)], 1u);
    __syncthreads();
    u32 c0, c1;                                  // bins from the top, two per thread
    {
        const int b0 = kBins - 1 - 2 * tid, b1 = b0 - 1;
        c0 = s_hist[b0];
        c1 = s_hist[b1];
        for (int q = 1; q < copies; ++q) { c0 += s_hist[q * kBins + b0]; c1 += s_hist[q * kBins + b1]; }
    }
    u32 S;
    const u32 incl = wg_incl_scan_u32<kListThreads>(c0 + c1, s_wave, &S);
    if (tid < R) {                               // the three ranks of every ranking
        u64 rk_k, rk_n;
        rank_of(tid / 3, &rk_k, &rk_n);
        const int which = tid % 3;               // upper bound, lower bound, estimate
        u32 want = 0, none = which == 0 ? 0x7FFFFFFFu : 0u;              // no such rank in the sample: unbounded
        if (rk_k == 0) {
            none = 0xFFFFFFFFu;
        } else if (S != 0) {
            const double p = static_cast<double>(rk_k) / static_cast<double>(rk_n);
            const double ks = p * static_cast<double>(S);
            const double sd = sqrt(static_cast<double>(kSampleUnit) * static_cast<double>(S) * p * (1.0 - p));
            const double m = (W == 1 ? static_cast<double>(w.margin16) / 16.0 * sd : 0.0) + 2.0;
            double r = which == 0 ? floor(ks - m) : (which == 1 ? ceil(ks + m) + 1.0 : floor(ks + 0.5));
            if (which == 2) r = r < 1.0 ? 1.0 : (r > static_cast<double>(S) ? static_cast<double>(S) : r);
            if (r >= 1.0 && r <= static_cast<double>(S)) want = static_cast<u32>(r);
        }
        s_want[tid] = want;
        s_key[tid] = none;
    }
    __syncthreads();
    {
        const u32 before = incl - c0 - c1;
        const u32 b0 = kBins - 1 - 2 * tid;
        for (int r = 0; r < R; ++r) {
            const u32 want = s_want[r];
            if (before < want && want <= incl) {
                const bool first = want <= before + c0;
                s_bin[r] = first ? b0 : b0 - 1;
                s_rem[r] = first ? want - before : want - before - c0;
            }
        }
    }
    __syncthreads();
    if (tid < R && s_want[tid]) {                // rankings that meet in a bin share its histogram: that of the first
        int f = 0;
        while (s_bin[f] != s_bin[tid]) ++f;
        if (f == tid) s_tab[s_bin[tid]] = static_cast<u8>(tid + 1);
    }
    constexpr int kShift2 = kShift0 - kBits2;
    for (int i = tid; i < R * kBins2; i += kListThreads) s_hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4 * kListUnits; ++i) {
        const u32 h = (valid & (1u << i)) ? s_tab[key[i] >> kShift0] : 0u;
        if (h) atomicAdd(&s_hist[(h - 1) * kBins2 + ((key[i] >> kShift2) & (kBins2 - 1))], 1u);
    }
    __syncthreads();
    for (int r = wave; r < R; r += kListThreads / 64) {
        if (s_want[r] == 0) continue;
        u32 bin = 0;
        if (wave_pick256(s_hist + (s_tab[s_bin[r]] - 1) * kBins2, s_rem[r], &bin)) {     // one lane
            const u32 key0 = (s_bin[r] << kShift0) | (bin << kShift2), low = (1u << kShift2) - 1u;
            s_key[r] = r % 3 == 0 ? key0 | low : (r % 3 == 1 ? key0 : key0 | ((low + 1u) >> 1));
        }
    }
    __syncthreads();
    if (tid < J) {
        const ListWin x = list_window(s_key[3 * tid], s_key[3 * tid + 1], s_key[3 * tid + 2]);
        if (W == 1) w.win[first_ranking + tid] = x;
        else        w.local[static_cast<u64>(at_local) * J + tid] = x;
        s_win[tid] = x;
    }
    if (W == 1 && J > 1) {
        __syncthreads();
        if (wave == 0) list_sort(s_win, J, s_want, w.sorted + first_ranking / J);
    }
}

// The sampling workgroups as a launch of their own.
template <bool LC, bool VEC>
__global__ __launch_bounds__(kListThreads) void k_list_sample(DataArgs a, ListArgs w) {
    const u32 g = a.per_tensor ? w.group_of[blockIdx.x] : 0u;
    const u64 r0 = static_cast<u64>(g) * a.J;
    const ListRank rk = w.rank[r0];
    const TensorDesc& tg = a.td[a.per_tensor ? g : 0];
    list_sample<LC, VEC>(w, a.J, a.mu, rk.n_groups, blockIdx.x - rk.group0, blockIdx.x, r0, a.per_tensor ? tg.chunk_start : 0,
                         a.per_tensor ? (tg.n + 3) / 4 : a.n_chunks * (kChunk / 4),
                         [&](u64 c) {
                             const TensorDesc& td = a.per_tensor ? tg : a.td[a.chunk_map[c]];
                             return SampleTensor{td.w, td.lam, td.n, td.chunk_start};
                         },
                         [&](int j, u64* k, u64* n) { *k = a.slots[r0 + j].k; *n = a.slots[r0 + j].n; });
}

// The sample as part of the launch that begins the call (few tensors): what the sampling workgroups need
// of the tables comes as kernel arguments, so they need not wait for the upload.  One launch less: 4 us.
constexpr int kBeginSampleTensors = 96;
struct BeginSampleArgs {
    UploadArgs up;
    uint4* zero;
    u64 n_zero;            // 16-byte words
    u32* chunk_map;
    u32 n_chunks;
    int n_tensors;
    u32 groups;            // sampling workgroups: the first of the grid
    int J;
    int per_tensor;
    float mu;
    u64 N;
    double density[kMaxJ];
    const float* w[kBeginSampleTensors];
    const float* lam[kBeginSampleTensors];
    u32 n[kBeginSampleTensors];
    u32 chunk_start[kBeginSampleTensors + 1];
    u16 group0[kBeginSampleTensors + 1];   // PER_TENSOR: first sampling workgroup of each tensor
};
static_assert(sizeof(BeginSampleArgs) + sizeof(ListArgs) <= 3584, "kernel arguments");
template <bool LC, bool VEC>
__global__ __launch_bounds__(kListThreads) void k_begin_sample(BeginSampleArgs b, ListArgs w) {
    __shared__ u32 s_start[kBeginSampleTensors + 1];
    const int tid = threadIdx.x;
    auto tensor_of_chunk_lds = [&](u32 c) {                // largest t with chunk_start[t] <= c
        int lo = 0, hi = b.n_tensors - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_start[mid] <= c) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    if (blockIdx.x == b.groups) {
        upload_words(b.up, tid, kListThreads);
        __syncthreads();                                   // every load has returned: its value went into a store
        if (tid == 0) store_ticket(b.up.done, b.up.ticket);
        return;
    }
    if (tid <= b.n_tensors) s_start[tid] = b.chunk_start[tid];
    if (blockIdx.x < b.groups) {
        __shared__ const float* s_w[kBeginSampleTensors];
        __shared__ const float* s_lam[kBeginSampleTensors];
        __shared__ u32 s_n[kBeginSampleTensors];
        if (tid < b.n_tensors) {
            s_w[tid] = b.w[tid];
            s_n[tid] = b.n[tid];
            if (LC) s_lam[tid] = b.lam[tid];
        }
        __syncthreads();
        u32 g = 0, W = b.groups, me = blockIdx.x;
        u64 first_chunk = 0, quads = static_cast<u64>(b.n_chunks) * (kChunk / 4), n_pop = b.N;
        if (b.per_tensor) {
            int lo = 0, hi = b.n_tensors - 1;              // the tensor this workgroup samples: the last with group0 <= its number
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (b.group0[mid] <= blockIdx.x) lo = mid; else hi = mid - 1;
            }
            g = static_cast<u32>(lo);
            W = static_cast<u32>(b.group0[g + 1]) - b.group0[g];
            me = blockIdx.x - b.group0[g];
            first_chunk = s_start[g];
            n_pop = s_n[g];
            quads = (n_pop + 3) / 4;
        }
        list_sample<LC, VEC>(w, b.J, b.mu, W, me, blockIdx.x, static_cast<u64>(g) * b.J, first_chunk, quads,
                             [&](u64 c) {
                                 const int t = b.per_tensor ? static_cast<int>(g) : tensor_of_chunk_lds(static_cast<u32>(c));
                                 return SampleTensor{s_w[t], LC ? s_lam[t] : nullptr, s_n[t], s_start[t]};
                             },
                             [&](int j, u64* k, u64* n) {  // as the host rounds: llround of the binary64 product, clamped
                                 const double x = b.density[j] * static_cast<double>(n_pop);
                                 const u64 kk = static_cast<u64>(llround(x));
                                 *k = kk > n_pop ? n_pop : kk;
                                 *n = n_pop;
                             });
        return;
    }
    __syncthreads();
    const u64 stride = static_cast<u64>(gridDim.x - b.groups - 1) * kListThreads;
    const u64 i0 = static_cast<u64>(blockIdx.x - b.groups - 1) * kListThreads + tid;
    const uint4 z = make_uint4(0, 0, 0, 0);
    for (u64 i = i0; i < b.n_zero; i += stride) b.zero[i] = z;
    for (u64 c = i0; c < b.n_chunks; c += stride) b.chunk_map[c] = static_cast<u32>(tensor_of_chunk_lds(static_cast<u32>(c)));
}

// Populations with several sampling workgroups, one workgroup here for each.  The workgroups' keys at the expected
// rank are as many independent draws around the threshold; order statistics W/2 -+ z sqrt(W)/2 of them bound its
// location with the confidence of z standard deviations, whatever their distribution.  A wavefront finds one order
// statistic bit by bit, with all W values in its registers.
constexpr int kBoundsThreads = 1024;
__global__ __launch_bounds__(kBoundsThreads) void k_list_bounds(DataArgs a, ListArgs w) {
    __shared__ u32 s_out[3 * kMaxJ];
    __shared__ ListWin s_win[kMaxJ];
    const u64 r0 = static_cast<u64>(blockIdx.x) * a.J;
    const ListRank rk = w.rank[r0];
    const u32 W = rk.n_groups, lane = threadIdx.x & 63u;
    if (W == 1) return;                          // its windows are written
    constexpr int kPer = kListMaxW / 64;
    const double d = static_cast<double>(w.margin16) / 16.0 * sqrt(static_cast<double>(W)) / 2.0;
    const u32 off = d >= static_cast<double>(W / 2) ? W / 2 : static_cast<u32>(ceil(d));
    for (u32 task = threadIdx.x >> 6; task < 3u * a.J; task += kBoundsThreads / 64) {
        const u32 j = task / 3, i = task % 3;    // i: upper bound, lower bound, estimate
        u32 v[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            v[q] = 0xFFFFFFFFu;                  // past the end: above every key (and every bound looked for)
            if (64 * q + lane < W) {
                const ListWin x = w.local[static_cast<u64>(rk.group0 + 64 * q + lane) * a.J + j];
                v[q] = i == 0 ? x.hi : (i == 1 ? x.lo : x.mid);
            }
        }
        const u32 pick = i == 0 ? (W / 2 + off < W ? W / 2 + off : W - 1) : (i == 1 ? (W / 2 - 1 >= off ? W / 2 - 1 - off : 0) : W / 2);
        u32 x = 0;                               // the largest x with at most `pick` values below it
        for (int bit = 31; bit >= 0; --bit) {
            const u32 cand = x | (1u << bit);
            u32 below = 0;
#pragma unroll
            for (int q = 0; q < kPer; ++q) below += static_cast<u32>(__popcll(__ballot(v[q] < cand)));
            if (below <= pick) x = cand;
        }
        if (lane == 0) s_out[task] = x;
    }
    __syncthreads();
    if (threadIdx.x < static_cast<u32>(a.J)) {
        const ListWin x = list_window(s_out[3 * threadIdx.x], s_out[3 * threadIdx.x + 1], s_out[3 * threadIdx.x + 2]);
        s_win[threadIdx.x] = x;
        w.win[r0 + threadIdx.x] = x;
    }
    if (a.J == 1) return;
    __syncthreads();
    if (threadIdx.x < 64) list_sort(s_win, a.J, s_out, w.sorted + blockIdx.x);
}

__device__ inline u32 lanes_below(u64 m) {       // set bits of m below this lane's
    return __builtin_amdgcn_mbcnt_hi(static_cast<u32>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<u32>(m), 0));
}

// ---- the one pass over the weights: one density ------------------------------------------------------------
//
// As k_window_fused, with one list per ranking and one counter update per wavefront (entries and keys above `mid` in
// the halves of a word).  One float4 per lane and array for the L-C forms, four for pruning (measured there).
template <bool LC, bool VEC, int QUADS, bool PQ>
__global__ __launch_bounds__(64) void k_list_sweep(DataArgs a, ListArgs w) {
    constexpr int kWaveElems = 256 * QUADS;
    constexpr u32 kSub = kChunk / kWaveElems;
    const u64 c = blockIdx.x / kSub;
    const u32 sub = blockIdx.x % kSub;
    if (c >= a.n_chunks) return;
    const int lane = threadIdx.x;
    const int t = static_cast<int>(a.chunk_map[c]);
    const TensorDesc& td = a.td[t];
    const u64 base = (c - td.chunk_start) * kChunk + static_cast<u64>(sub) * kWaveElems;
    const u64 n = td.n;
    if (base >= n) return;
    const u32 r = a.per_tensor ? static_cast<u32>(t) : 0u;
    const ListWin win = w.win[r];
    const u32 lo = win.lo, span = win.hi - win.lo, mid = win.mid;
    OutDesc o{};
    if (w.write) o = w.out[t];
    const float mu = a.mu;
    const bool full = VEC && base + kWaveElems <= n;                    // uniform over the wavefront

    float wk[QUADS][4], lk[QUADS][4];
    if (full) {
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            const float4 x = ld4_stream(td.w + base + q * 256 + lane * 4);
            wk[q][0] = x.x; wk[q][1] = x.y; wk[q][2] = x.z; wk[q][3] = x.w;
            if (LC) {
                const float4 y = ld4_stream(td.lam + base + q * 256 + lane * 4);
                lk[q][0] = y.x; lk[q][1] = y.y; lk[q][2] = y.z; lk[q][3] = y.w;
            }
        }
    }
    u32 key[QUADS][4];
    u64 in_window[QUADS][4];                                            // lanes whose element is inside the window
    u32 total = 0, kept = 0, nz = 0;                                    // sums over the wavefront
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        const u64 e0 = base + static_cast<u64>(q) * 256 + lane * 4;
        if (!full) {
#pragma unroll
            for (int k = 0; k < 4; ++k) { wk[q][k] = 0.0f; lk[q][k] = 0.0f; }
            if (e0 < n) {
                load4<VEC>(td.w, e0, n, wk[q]);
                if (LC) load4<VEC>(td.lam, e0, n, lk[q]);
            }
        }
        float th[4], ln[4], gr[4];
        u8 m[4];
        u16 h16[4] = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float v = LC ? lc_shift(wk[q][k], lk[q][k], mu) : wk[q][k];
            const u32 x = mag_key(v);
            key[q][k] = x;
            const bool in = full || e0 + k < n;
            const bool keep = x >= mid;                                 // final outside the window, provisional inside
            kept += static_cast<u32>(__popcll(__ballot(keep && in)));
            in_window[q][k] = __ballot(in && x - lo <= span);
            total += static_cast<u32>(__popcll(in_window[q][k]));
            m[k] = keep ? 1 : 0;
            th[k] = keep ? v : 0.0f;
            if (PQ) {
                h16[k] = f32_to_f16_rne(th[k]);
                th[k] = f16_bits_to_f32(h16[k]);
                nz += static_cast<u32>(__popcll(__ballot(in && (h16[k] & 0x7FFFu) != 0)));
            }
            if (LC) {
                const float e = __fsub_rn(wk[q][k], th[k]);
                const float p = __fmul_rn(mu, e);
                ln[k] = __fsub_rn(lk[q][k], p);
                gr[k] = __fsub_rn(p, ln[k]);
            }
        }
        if (full) {
            if (o.theta) st4_stream(o.theta + e0, th[0], th[1], th[2], th[3]);
            if (!LC && o.theta16)
                st_code4_stream(o.theta16 + e0, f32_to_f16_rne(th[0]), f32_to_f16_rne(th[1]), f32_to_f16_rne(th[2]), f32_to_f16_rne(th[3]));
            if (PQ && o.theta16) st_code4_stream(o.theta16 + e0, h16[0], h16[1], h16[2], h16[3]);
            if (LC && w.write) {
                st4_stream(td.lam_out + e0, ln[0], ln[1], ln[2], ln[3]);
                if (td.grad) st4_stream(td.grad + e0, gr[0], gr[1], gr[2], gr[3]);
            }
            if (o.mask) st_mask4_stream(o.mask + e0, m[0], m[1], m[2], m[3]);
        } else if (e0 < n) {
            if (o.theta) store4<VEC>(o.theta, e0, n, th);
            if (!LC && o.theta16) {
                u16 h[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) h[k] = f32_to_f16_rne(th[k]);
                store4_u16<VEC>(o.theta16, e0, n, h);
            }
            if (PQ && o.theta16) store4_u16<VEC>(o.theta16, e0, n, h16);
            if (LC && w.write) {
                store4<VEC>(td.lam_out, e0, n, ln);
                if (td.grad) store4<VEC>(td.grad, e0, n, gr);
            }
            if (o.mask) store4_u8<VEC>(o.mask, e0, n, m);
        }
    }
    const ListRank rk = w.rank[r];
    const u32 seg = blockIdx.x % rk.n_segs;
    if (PQ && lane == 1 && nz) atomicAdd(&w.nnz[seg], nz);
    if ((total | kept) == 0) return;
    u64 b = 0;
    if (lane == 0)
        b = atomicAdd(reinterpret_cast<unsigned long long*>(&w.cnt[static_cast<u64>(r) * w.max_segs + seg]),
                      (static_cast<unsigned long long>(kept) << 32) | total);
    if (total == 0) return;
    u32 pos = __shfl(static_cast<u32>(b), 0, 64);
    const u64 first = rk.base + static_cast<u64>(seg) * rk.seg_cap;
    const u32 i0 = static_cast<u32>(c) * kChunk + sub * kWaveElems + lane * 4;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u64 m = in_window[q][k];
            if (m == 0) continue;                                       // uniform
            const u32 at = pos + lanes_below(m);
            if (((m >> lane) & 1u) && at < rk.seg_cap) {
                w.key[first + at] = key[q][k];
                w.idx[first + at] = i0 + q * 256 + k;
            }
            pos += static_cast<u32>(__popcll(m));
        }
    }
}

// ---- the one pass over the weights: several densities --------------------------------------------------------
//
// The keys of 1024 elements sit in the registers of a wavefront.  Their regions (ListSorted: one compare and add per
// key and ranking) give the masks of all rankings by byte arithmetic, four elements at a time: bit 7 of region + bias.
// The few keys inside a window are gathered in LDS; the counter updates of all rankings are then one instruction (lane j
// updates ranking j), so their latency is paid once, and the entries leave in runs.  Masks alone leave as 16 bytes per
// lane, the regions having changed places in LDS.
constexpr int kListMultiQuads = 4;
// Calls of few weights take a quarter of that per wavefront: each ranking costs a wavefront some 3 us of latency (ten
// densities of 46 thousand weights 66 us with 1024 elements to a wavefront, 45.9 with 256; of 295 thousand 67.5
// and 53.7; two of 295 thousand 37.4 and 36.9, of 2.3 M 42.3 and 47.5).
constexpr u64 kListMultiFew = static_cast<u64>(1) << 19;
__host__ __device__ inline int list_multi_quads(u64 N) { return N <= kListMultiFew ? 1 : kListMultiQuads; }
constexpr u32 kListMultiBuf = 512;               // buffered entries of a wavefront: an equal share for each ranking; with more, they come from the tile
struct ListMultiShared {
    u32 key[kListMultiBuf];
    u32 tile[256 * kListMultiQuads];             // the tile's keys, then its regions
    u32 count[kMaxJ];
    u32 gap[2 * (kMaxJ + 1)];
    u32 ranking[kMaxJ];
    u16 off[kListMultiBuf];
};

__device__ inline u32 list_reserve(const ListArgs& w, u64 r, const ListRank& rk, u32 count, u32 kept) {
    return static_cast<u32>(atomicAdd(reinterpret_cast<unsigned long long*>(&w.cnt[r * w.max_segs + blockIdx.x % rk.n_segs]),
                                      (static_cast<unsigned long long>(kept) << 32) | count));
}
// `mine`: in lane j, ranking j's buffered entries and (upper half) its keys from the estimate on.
__device__ inline void list_multi_flush(const DataArgs& a, const ListArgs& w, const ListMultiShared& sh, u64 r0, u64 mine, u32 i0) {
    const int lane = threadIdx.x;
    ListRank rk{};
    u32 at = 0;
    if (lane < a.J && mine) {
        rk = w.rank[r0 + lane];
        at = list_reserve(w, r0 + lane, rk, static_cast<u32>(mine), static_cast<u32>(mine >> 32));
    }
    const u64 first = rk.base + (rk.n_segs ? static_cast<u64>(blockIdx.x % rk.n_segs) * rk.seg_cap : 0);
    const u32 share = kListMultiBuf / static_cast<u32>(a.J);
    __syncthreads();                                                    // one wavefront: orders the LDS buffer
    for (int j = 0; j < a.J; ++j) {
        const u32 count = __shfl(static_cast<u32>(mine), j, 64);
        const u32 pos = __shfl(at, j, 64), cap = __shfl(rk.seg_cap, j, 64);
        const u64 to = ((static_cast<u64>(__shfl(static_cast<u32>(first >> 32), j, 64)) << 32) | __shfl(static_cast<u32>(first), j, 64)) + pos;
        for (u32 i = lane; i < count; i += 64)
            if (pos + i < cap) {
                w.key[to + i] = sh.key[j * share + i];
                w.idx[to + i] = i0 + sh.off[j * share + i];
            }
    }
}

// The general form: a tile that is ragged, or windows that overlap.  The rankings are walked one by one.
template <bool VEC, int Q>
__device__ inline void list_multi_general(const DataArgs& a, const ListArgs& w, ListMultiShared& sh, const TensorDesc& td, int t, u64 c, u32 sub,
                                          u64 base, bool full) {
    constexpr int kWaveElems = 256 * Q;
    const int lane = threadIdx.x;
    const u64 n = td.n;
    const u64 r0 = a.per_tensor ? static_cast<u64>(t) * a.J : 0;
    float v[Q][4];
    u32 in = 0xFFFFFFFFu;                                               // bit q * 4 + k: the element exists
    if (full) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const float4 x = *reinterpret_cast<const float4*>(td.w + base + q * 256 + lane * 4);
            v[q][0] = x.x; v[q][1] = x.y; v[q][2] = x.z; v[q][3] = x.w;
        }
    } else {
        in = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const u64 e0 = base + static_cast<u64>(q) * 256 + lane * 4;
            v[q][0] = v[q][1] = v[q][2] = v[q][3] = 0.0f;
            if (e0 < n) {
                load4<VEC>(td.w, e0, n, v[q]);
                const u32 have = n - e0 < 4 ? static_cast<u32>(n - e0) : 4u;
                in |= ((1u << have) - 1u) << (4 * q);
            }
        }
    }
    const u32 i0 = static_cast<u32>(c) * kChunk + sub * kWaveElems;
    const u32 share = kListMultiBuf / static_cast<u32>(a.J);
    u64 mine = 0;                                                       // lane j: ranking j's buffered entries and kept keys
    for (int j = 0; j < a.J; ++j) {
        const ListWin win = w.win[r0 + j];
        const u32 lo = win.lo, span = win.hi - win.lo, mid = win.mid;
        OutDesc o{};
        if (w.write) o = w.out[static_cast<u64>(j) * a.n_tensors + t];
        u32 count = 0, kept = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const u64 e0 = base + static_cast<u64>(q) * 256 + lane * 4;
            u8 m[4];
            float th[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u32 x = mag_key(v[q][k]);
                const bool there = full || ((in >> (4 * q + k)) & 1u);
                const bool keep = x >= mid;
                kept += static_cast<u32>(__popcll(__ballot(keep && there)));
                m[k] = keep ? 1 : 0;
                th[k] = keep ? v[q][k] : 0.0f;
                const u64 hit = __ballot(there && x - lo <= span);
                if (hit != 0) {                                         // uniform
                    const u32 n_hit = static_cast<u32>(__popcll(hit));
                    const bool me = (hit >> lane) & 1u;
                    if (count + n_hit <= share) {
                        if (me) {
                            sh.key[j * share + count + lanes_below(hit)] = x;
                            sh.off[j * share + count + lanes_below(hit)] = static_cast<u16>(q * 256 + lane * 4 + k);
                        }
                        count += n_hit;
                    } else {                                            // full buffer: straight to the list
                        const ListRank rk = w.rank[r0 + j];
                        u32 at = 0;
                        if (lane == 0) at = list_reserve(w, r0 + j, rk, n_hit, 0);
                        at = __shfl(at, 0, 64) + lanes_below(hit);
                        if (me && at < rk.seg_cap) {
                            const u64 to = rk.base + static_cast<u64>(blockIdx.x % rk.n_segs) * rk.seg_cap + at;
                            w.key[to] = x;
                            w.idx[to] = i0 + q * 256 + lane * 4 + k;
                        }
                    }
                }
            }
            if (full) {
                if (o.mask) st_mask4_stream(o.mask + e0, m[0], m[1], m[2], m[3]);
                if (o.theta) st4_stream(o.theta + e0, th[0], th[1], th[2], th[3]);
                if (o.theta16)
                    st_code4_stream(o.theta16 + e0, f32_to_f16_rne(th[0]), f32_to_f16_rne(th[1]), f32_to_f16_rne(th[2]), f32_to_f16_rne(th[3]));
            } else if (e0 < n) {
                if (o.mask) store4_u8<VEC>(o.mask, e0, n, m);
                if (o.theta) store4<VEC>(o.theta, e0, n, th);
                if (o.theta16) {
                    u16 h[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) h[k] = f32_to_f16_rne(th[k]);
                    store4_u16<VEC>(o.theta16, e0, n, h);
                }
            }
        }
        if (lane == j) mine = (static_cast<u64>(kept) << 32) | count;
    }
    list_multi_flush(a, w, sh, r0, mine, i0);
}

// WIDE: masks only, each 16-byte aligned.
template <bool VEC, bool WIDE, int Q>
__global__ __launch_bounds__(64) void k_list_sweep_multi(DataArgs a, ListArgs w) {
    constexpr int kWaveElems = 256 * Q;
    constexpr u32 kSub = kChunk / kWaveElems;
    __shared__ __align__(16) ListMultiShared sh;
    const u64 c = blockIdx.x / kSub;
    const u32 sub = blockIdx.x % kSub;
    if (c >= a.n_chunks) return;
    const int lane = threadIdx.x;
    const int t = static_cast<int>(a.chunk_map[c]);
    const TensorDesc& td = a.td[t];
    const u64 base = (c - td.chunk_start) * kChunk + static_cast<u64>(sub) * kWaveElems;
    if (base >= td.n) return;
    const u64 r0 = a.per_tensor ? static_cast<u64>(t) * a.J : 0;
    const bool full = VEC && base + kWaveElems <= td.n;                 // uniform over the wavefront
    const ListSorted& srt = w.sorted[a.per_tensor ? t : 0];
    if (!full || !srt.disjoint) {
        list_multi_general<VEC, Q>(a, w, sh, td, t, c, sub, base, full);
        return;
    }
    float v[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const float4 x = *reinterpret_cast<const float4*>(td.w + base + q * 256 + lane * 4);
        v[q][0] = x.x; v[q][1] = x.y; v[q][2] = x.z; v[q][3] = x.w;
    }
    const u32 n = srt.n;
    if (lane < kMaxJ) { sh.count[lane] = 0; sh.ranking[lane] = srt.ranking[lane]; }
    if (lane <= kMaxJ) { sh.gap[2 * lane] = srt.gap_lo[lane]; sh.gap[2 * lane + 1] = srt.gap_len[lane]; }
    u32 region[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) region[q][k] = 0;
    for (u32 p = 0; p < n; ++p) {
        const u32 mid = srt.mid[p];                                     // uniform
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) region[q][k] += mag_key(v[q][k]) >= mid ? 1u : 0u;
    }
    __syncthreads();                                                    // one wavefront: orders LDS
    // the keys inside a window: a bit per element, then every lane takes its own one after the other
    u32 inside = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        *reinterpret_cast<uint4*>(&sh.tile[q * 256 + lane * 4]) = make_uint4(mag_key(v[q][0]), mag_key(v[q][1]), mag_key(v[q][2]), mag_key(v[q][3]));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint2 gap = *reinterpret_cast<const uint2*>(&sh.gap[2 * region[q][k]]);
            if (mag_key(v[q][k]) - gap.x >= gap.y) inside |= 1u << (4 * q + k);
        }
    }
    u32 packed[Q];                                                      // regions of a float4's elements, a byte each
#pragma unroll
    for (int q = 0; q < Q; ++q) packed[q] = region[q][0] | (region[q][1] << 8) | (region[q][2] << 16) | (region[q][3] << 24);
    const u32 i0 = static_cast<u32>(c) * kChunk + sub * kWaveElems, share = kListMultiBuf / static_cast<u32>(a.J);
    bool full_buffer = false;
    while (inside) {
        const u32 i = static_cast<u32>(__ffs(inside)) - 1u, off = (i >> 2) * 256 + lane * 4 + (i & 3u);
        inside &= inside - 1u;
        u32 word = packed[0];
#pragma unroll
        for (int q = 1; q < Q; ++q) word = (i >> 2) == static_cast<u32>(q) ? packed[q] : word;
        const u32 r = (word >> (8 * (i & 3u))) & 0xFFu, x = sh.tile[off];
        // below the gap of its region: the window of the highest estimate it reaches; else the next one up
        const u32 j = sh.ranking[x < sh.gap[2 * r] ? n - r : n - r - 1u];
        const u32 at = atomicAdd(&sh.count[j], 1u);
        if (at < share) {
            sh.key[j * share + at] = x;
            sh.off[j * share + at] = static_cast<u16>(off);
        }
        full_buffer = full_buffer || at >= share;
    }
    u64 full_buffers = __ballot(full_buffer);
    if (full_buffers != 0) full_buffers = __ballot(lane < a.J && sh.count[lane < a.J ? lane : 0] > share);
    while (full_buffers != 0) {                                         // uniform.  All of that ranking's entries from the tile,
        const u32 j = static_cast<u32>(__ffsll(static_cast<long long>(full_buffers))) - 1u;            // with one reservation
        full_buffers &= full_buffers - 1u;
        const ListWin win = w.win[r0 + j];
        const ListRank rk = w.rank[r0 + j];
        u32 pos = 0;
        if (lane == 0) pos = list_reserve(w, r0 + j, rk, sh.count[j], 0);
        pos = __shfl(pos, 0, 64);
        const u64 first = rk.base + static_cast<u64>(blockIdx.x % rk.n_segs) * rk.seg_cap;
        for (u32 off = lane; off < static_cast<u32>(kWaveElems); off += 64) {
            const u32 x = sh.tile[off];
            const bool me = x - win.lo <= win.hi - win.lo;
            const u64 m = __ballot(me);
            const u32 at = pos + lanes_below(m);
            if (me && at < rk.seg_cap) { w.key[first + at] = x; w.idx[first + at] = i0 + off; }
            pos += static_cast<u32>(__popcll(m));
        }
    }
    if constexpr (WIDE) {                                               // lane l takes the regions of elements 16 l .. 16 l + 15
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) sh.tile[q * 64 + lane] = packed[q];
        __syncthreads();
        const uint4 x = *reinterpret_cast<const uint4*>(&sh.tile[4 * lane]);
        packed[0] = x.x; packed[1] = x.y; packed[2] = x.z; packed[3] = x.w;
    }
    u32 kept_of_lane = 0;                                               // lane j: ranking j's keys from its estimate on
    for (int j = 0; j < a.J; ++j) {
        const u32 bias = srt.bias[j] * 0x01010101u;                     // uniform
        OutDesc o{};
        if (w.write) o = w.out[static_cast<u64>(j) * a.n_tensors + t];
        u32 m[Q], kept = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            m[q] = ((packed[q] + bias) >> 7) & 0x01010101u;
            kept = __builtin_amdgcn_udot4(m[q], 0x01010101u, kept, false);
        }
        if constexpr (WIDE) {
            if (o.mask) {
                u32x4 t4;
                t4.x = m[0]; t4.y = m[1]; t4.z = m[2]; t4.w = m[3];
                st_words4_stream(o.mask + base + lane * 16, t4);
            }
        } else {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const u64 e0 = base + q * 256 + lane * 4;
                if (o.mask) st_mask4_stream(o.mask + e0, static_cast<u8>(m[q] & 1u), static_cast<u8>((m[q] >> 8) & 1u),
                                            static_cast<u8>((m[q] >> 16) & 1u), static_cast<u8>(m[q] >> 24));
                if (!o.theta && !o.theta16) continue;
                float th[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) th[k] = ((m[q] >> (8 * k)) & 1u) ? v[q][k] : 0.0f;
                if (o.theta) st4_stream(o.theta + e0, th[0], th[1], th[2], th[3]);
                if (o.theta16)
                    st_code4_stream(o.theta16 + e0, f32_to_f16_rne(th[0]), f32_to_f16_rne(th[1]), f32_to_f16_rne(th[2]), f32_to_f16_rne(th[3]));
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) kept += __shfl_xor(kept, d, 64);
        if (lane == j) kept_of_lane = kept;
    }
    __syncthreads();
    const u32 buffered = lane < a.J && sh.count[lane] <= share ? sh.count[lane] : 0u;
    list_multi_flush(a, w, sh, r0, (static_cast<u64>(kept_of_lane) << 32) | buffered, i0);
}

// ---- the threshold among the listed keys ---------------------------------------------------------------

// f(there, key, entry) for the entries of ranking s that this wavefront takes: every `stride`-th segment, kListDeep rows
// of four segments at a time (their loads in flight together); called by all lanes, `there` says which hold an entry.
constexpr u32 kListDeep = 4;
template <typename F>
__device__ inline void list_walk(const ListArgs& w, u32 s, const ListRank& rk, u32 first_seg, u32 stride, F&& f) {
    const u32 lane = threadIdx.x & 63u;
    for (u32 seg0 = first_seg; seg0 < rk.n_segs; seg0 += 64 * stride) {
        const u32 my_seg = seg0 + lane * stride;
        u32 my_cnt = my_seg < rk.n_segs ? static_cast<u32>(w.cnt[static_cast<u64>(s) * w.max_segs + my_seg]) : 0u;
        if (my_cnt > rk.seg_cap) my_cnt = rk.seg_cap;
        for (u32 l = 0; l < 64 && seg0 + l * stride < rk.n_segs; l += 4) {
            u32 cnt[4], most = 0;
            u64 first[4];
#pragma unroll
            for (u32 b = 0; b < 4; ++b) {
                cnt[b] = __shfl(my_cnt, static_cast<int>(l + b), 64);
                first[b] = rk.base + static_cast<u64>(seg0 + (l + b) * stride) * rk.seg_cap;
                most = cnt[b] > most ? cnt[b] : most;
            }
            for (u32 i0 = 0; i0 < most; i0 += 64 * kListDeep) {
                u32 x[kListDeep][4];
#pragma unroll
                for (u32 d = 0; d < kListDeep; ++d)
#pragma unroll
                    for (u32 b = 0; b < 4; ++b) {
                        const u32 i = i0 + 64 * d + lane;
                        x[d][b] = i < cnt[b] ? w.key[first[b] + i] : 0u;
                    }
#pragma unroll
                for (u32 d = 0; d < kListDeep; ++d)
#pragma unroll
                    for (u32 b = 0; b < 4; ++b) {
                        const u32 i = i0 + 64 * d + lane;
                        if (i0 + 64 * d < cnt[b]) f(i < cnt[b], x[d][b], first[b] + i);           // uniform
                    }
            }
        }
    }
}

// Counts of a ranking's listed keys per bin of its window; `parts` workgroups per ranking.
__global__ __launch_bounds__(kBlock) void k_list_hist(DataArgs a, ListArgs w) {
    __shared__ u32 s_hist[kListBins];
    const u32 s = blockIdx.x / w.parts, part = blockIdx.x % w.parts;
    const ListRank rk = w.rank[s];
    const ListWin win = w.win[s];
    const u32 wave = threadIdx.x >> 6, first = part * (kBlock / 64) + wave, stride = w.parts * (kBlock / 64);
    if (part * (kBlock / 64) >= rk.n_segs) return;         // uniform: nothing for this workgroup
    s_hist[threadIdx.x] = 0;                               // kListBins == kBlock
    __syncthreads();
    const u32 lo = win.lo, shift = win.bins & 0xFFu;
    list_walk(w, s, rk, first, stride, [&](bool there, u32 key, u64) {
        if (there) atomicAdd(&s_hist[(key - lo) >> shift], 1u);
    });
    __syncthreads();
    const u32 v = s_hist[threadIdx.x];
    if (v) atomicAdd(&w.hist[static_cast<u64>(s) * kListBins + threadIdx.x], v);
}

// The outputs of up to B listed elements, with the decision each should have had.  The dependent loads of the elements
// (tensor, its pointers, the inputs) are issued side by side: one after the other they take some 3 us an element.
template <bool LC, bool PQ, int B>
__device__ inline void list_fix(const DataArgs& a, const ListArgs& w, u32 j, const u32 (&idx)[B], const bool (&keep)[B], const bool (&on)[B], int* nz) {
    u32 t[B];
#pragma unroll
    for (int b = 0; b < B; ++b) t[b] = on[b] ? a.chunk_map[idx[b] / kChunk] : 0u;
    const float* wp[B];
    const float* lp[B];
    float* lo[B];
    float* gr[B];
    u64 e[B];
    OutDesc o[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const TensorDesc& td = a.td[t[b]];
        wp[b] = td.w;
        if (LC) { lp[b] = td.lam; lo[b] = td.lam_out; gr[b] = td.grad; }
        e[b] = static_cast<u64>(idx[b]) - td.chunk_start * kChunk;
        o[b] = w.out[static_cast<u64>(j) * a.n_tensors + t[b]];
    }
    float wv[B], lv[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        wv[b] = on[b] ? wp[b][e[b]] : 0.0f;
        lv[b] = LC && on[b] ? lp[b][e[b]] : 0.0f;
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        if (!on[b]) continue;
        if (LC) {
            const float x = lc_shift(wv[b], lv[b], a.mu);
            float th = keep[b] ? x : 0.0f;
            if (PQ) {
                const u16 hv = f32_to_f16_rne(x), h = keep[b] ? hv : static_cast<u16>(0);
                th = f16_bits_to_f32(h);
                if (o[b].theta16) o[b].theta16[e[b]] = h;
                if ((hv & 0x7FFFu) != 0) *nz += keep[b] ? 1 : -1;
            }
            const float p = __fmul_rn(a.mu, __fsub_rn(wv[b], th));
            const float ln = __fsub_rn(lv[b], p);
            if (o[b].theta) o[b].theta[e[b]] = th;
            lo[b][e[b]] = ln;
            if (gr[b]) gr[b][e[b]] = __fsub_rn(p, ln);
        } else {
            const float th = keep[b] ? wv[b] : 0.0f;
            if (o[b].theta) o[b].theta[e[b]] = th;
            if (o[b].theta16) o[b].theta16[e[b]] = f32_to_f16_rne(th);
        }
        if (o[b].mask) o[b].mask[e[b]] = keep[b] ? 1 : 0;
    }
}
template <bool LC, bool PQ>
__device__ inline void list_fix_one(const DataArgs& a, const ListArgs& w, u32 j, u32 idx, bool keep, int* nz) {
    const u32 i1[1] = {idx};
    const bool k1[1] = {keep}, on1[1] = {true};
    list_fix<LC, PQ, 1>(a, w, j, i1, k1, on1, nz);
}
// Places in an LDS queue for the lanes that want one: one update of its counter per wavefront.
__device__ inline u32 wave_push(u32* counter, bool wanted) {
    const u64 m = __ballot(wanted);
    u32 at = 0;
    if (m != 0) {                                          // uniform
        const int leader = __ffsll(static_cast<long long>(m)) - 1;
        if (static_cast<int>(threadIdx.x & 63u) == leader) at = atomicAdd(counter, static_cast<u32>(__popcll(m)));
        at = __shfl(at, leader, 64);
    }
    return at + lanes_below(m);
}

// The queued wrong decisions of a workgroup: entry of the ranking's list, top bit = the right decision.
template <bool LC, bool PQ, int THREADS>
__device__ inline void list_fix_queue(const DataArgs& a, const ListArgs& w, u32 j, const u32* __restrict__ ids, const u32* queue, u32 n_q, int* nz) {
    constexpr int B = 4;
    for (u32 q0 = threadIdx.x; q0 < n_q; q0 += THREADS * B) {
        u32 idx[B];
        bool keep[B], on[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const u32 q = q0 + b * THREADS;
            on[b] = q < n_q;
            const u32 v = on[b] ? queue[q] : 0u;
            keep[b] = (v >> 31) != 0;
            idx[b] = on[b] ? ids[v & 0x7FFFFFFFu] : 0u;
        }
        list_fix<LC, PQ, B>(a, w, j, idx, keep, on, nz);
    }
}

// Every workgroup finds the bin of rank k - above from the counts.  Elements in the bins beside it are settled here:
// wrong decisions are queued in LDS, so that their chains of dependent loads run side by side.
template <bool LC, bool PQ>
__global__ __launch_bounds__(kBlock) void k_list_gather(DataArgs a, ListArgs w) {
    constexpr u32 kQueue = 2048;
    __shared__ u64 s_wave[kBlock / 64];
    constexpr u32 kFound = 1024;
    __shared__ u32 s_queue[kQueue];                        // wrong decisions: entry, top bit = the right one
    __shared__ u32 s_fkey[kFound], s_fidx[kFound];         // entries in the bin (one reservation per workgroup: updates of
                                                           // one counter that return a value take turns)
    __shared__ u32 s_over, s_gtmid, s_bin, s_want, s_in, s_n, s_f, s_base;
    const u32 s = blockIdx.x / w.parts, part = blockIdx.x % w.parts, tid = threadIdx.x, lane = tid & 63u;
    const ListRank rk = w.rank[s];
    const ListWin win = w.win[s];
    const Slot& slot = a.slots[s];
    if (part != 0 && part * (kBlock / 64) >= rk.n_segs) return;          // uniform
    if (PQ && w.nnz_out && w.write && part == 0) {         // the sweep's count of non-zero codes, corrected by k_list_settle
        u64 v = 0, total;
        for (u32 i = tid; i < static_cast<u32>(kListSegs); i += kBlock) v += w.nnz[i];
        block_excl_scan_u64(v, s_wave, &total);
        if (tid == 0) *w.nnz_out = total;
    }
    if (slot.state != kSelecting) {                        // k == 0: nothing listed
        if (part == 0 && tid == 0) w.bin_want[s] = 0;
        return;
    }
    if (tid == 0) { s_over = 0; s_n = 0; s_f = 0; s_in = 0; s_want = 0; }
    __syncthreads();
    u64 cnt = 0;
    for (u32 seg = tid; seg < rk.n_segs; seg += kBlock) {
        const u64 v = w.cnt[static_cast<u64>(s) * w.max_segs + seg];
        if (static_cast<u32>(v) > rk.seg_cap) s_over = 1;
        cnt += v;                                          // both halves: neither sum reaches 2^32
    }
    const u32 bin_of_tid = kListBins - 1 - tid;            // kListBins == kBlock: bins from the top
    const u32 h = w.hist[static_cast<u64>(s) * kListBins + bin_of_tid];
    u64 sums, listed;
    block_excl_scan_u64(cnt, s_wave, &sums);
    const u64 higher = block_excl_scan_u64(h, s_wave, &listed);
    const u32 shift = win.bins & 0xFFu, mid_bin = win.bins >> 8;
    if (bin_of_tid == mid_bin) s_gtmid = static_cast<u32>(higher) + h;
    __syncthreads();
    const u64 above = (sums >> 32) - s_gtmid;              // keys above the window
    const u64 want = slot.k - above;
    if (above < slot.k && higher < want && want <= higher + h) { s_bin = bin_of_tid; s_want = static_cast<u32>(want - higher); s_in = h; }
    __syncthreads();
    const bool ok = s_over == 0 && s_want != 0 && s_in <= w.gather_cap;
    if (part == 0 && tid == 0) {
        w.bin_want[s] = ok ? s_want : 0;
        if (!ok) w.fail_list[atomicAdd(&w.fb->failed, 1u)] = s;
    }
    if (!ok) return;                                       // uniform over all workgroups of the ranking
    const u32 lo = win.lo, bin = s_bin;
    const u32 g = s / a.J, j = s - g * a.J;
    int nz = 0;
    u32* gkey = w.gkey + static_cast<u64>(s) * w.gather_cap;
    u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
    list_walk(w, s, rk, part * (kBlock / 64) + (tid >> 6), w.parts * (kBlock / 64), [&](bool there, u32 key, u64 at) {
        const u32 b = (key - lo) >> shift;
        const bool found = there && b == bin, wrong = w.write && there && b != bin && (b > bin) != (b >= mid_bin);
        const u32 f = wave_push(&s_f, found);
        if (found) {
            if (f < kFound) {
                s_fkey[f] = key;
                s_fidx[f] = static_cast<u32>(at - rk.base);
            } else {                                       // a full buffer: straight to the list
                const u32 to = atomicAdd(&w.gathered[s], 1u);
                if (to < w.gather_cap) { gkey[to] = key; gidx[to] = w.idx[at]; }
            }
        }
        const u32 q = wave_push(&s_n, wrong);
        if (wrong) {
            if (q < kQueue) s_queue[q] = static_cast<u32>(at - rk.base) | (b > bin ? 0x80000000u : 0u);
            else            list_fix_one<LC, PQ>(a, w, j, w.idx[at], b > bin, &nz);
        }
    });
    __syncthreads();
    const u32 n_f = s_f < kFound ? s_f : kFound, n_q = s_n < kQueue ? s_n : kQueue;
    if (tid == 0 && n_f) s_base = atomicAdd(&w.gathered[s], n_f);
    list_fix_queue<LC, PQ, kBlock>(a, w, j, w.idx + rk.base, s_queue, n_q, &nz);
    __syncthreads();
    for (u32 f = tid; f < n_f; f += kBlock) {
        const u32 to = s_base + f;
        if (to < w.gather_cap) { gkey[to] = s_fkey[f]; gidx[to] = w.idx[rk.base + s_fidx[f]]; }
    }
    if (PQ) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) nz += __shfl_xor(nz, d, 64);
        if (lane == 0 && nz != 0)
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.ctl->nnz_delta), static_cast<unsigned long long>(static_cast<long long>(nz)));
    }
}

// ---- settle -----------------------------------------------------------------------------------------------------

__device__ inline condensa_select select_record(const Slot& slot, bool ranked, u64 T, u64 keep_ties, u64 n_tie, u64 tie_end, u64 path) {
    condensa_select out;
    out.n = slot.n;
    out.k = slot.k;
    out.n_gt = ranked ? slot.k - keep_ties : 0;
    out.n_tie_kept = ranked ? keep_ties : 0;
    out.n_tie = ranked ? n_tie : 0;
    out.threshold_key = ranked ? T : ~static_cast<u64>(0);
    out.tie_end = ranked ? tie_end : 0;
    out.path = path;
    return out;
}

constexpr u32 kListPairs = 256;                  // entries ranked by comparing all pairs
struct ListShared {        // LDS of list_rank
    u32 key[kListRanked], idx[kListRanked];      // the gathered entries, when they fit
    u32 pkey[kListPairs], pidx[kListPairs];
    __align__(16) u32 hist[kListBins];
    u32 wave[kListThreads / 64];
    u32 T, r, n_tie, last, pick, rem, n;
};

// The bin of sh.hist that holds rank r (from the top, or from the bottom), the rank inside it and its count.
__device__ inline void list_pick(ListShared& sh, bool from_top, u32 r, u32* bin, u32* rem, u32* count) {
    if (threadIdx.x < 64) {
        const u32 lane = threadIdx.x;
        const uint4 c4 = *reinterpret_cast<const uint4*>(sh.hist + (from_top ? 252 - 4 * lane : 4 * lane));
        const u32 c[4] = {from_top ? c4.w : c4.x, from_top ? c4.z : c4.y, from_top ? c4.y : c4.z, from_top ? c4.x : c4.w};
        u32 incl = c[0] + c[1] + c[2] + c[3];
        const u32 sum = incl;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const u32 up = __shfl_up(incl, d, 64);
            if (static_cast<int>(lane) >= d) incl += up;
        }
        u32 before = incl - sum;
        if (before < r && r <= incl) {
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
                if (before < r && r <= before + c[i]) {
                    sh.pick = from_top ? 255 - 4 * lane - i : 4 * lane + i;
                    sh.rem = r - before;
                    sh.n = c[i];
                }
                before += c[i];
            }
        }
    }
    __syncthreads();
    *bin = sh.pick;
    *rem = sh.rem;
    *count = sh.n;
    __syncthreads();
}

// One workgroup: the element at rank `want` of the gathered ones (key descending, then index ascending) is the last
// one kept; state, record and the outputs of gathered elements whose decision was wrong.  One more counting level leaves
// a handful, which are ranked by comparing all pairs.
// `want` 0: the ranking failed.  `n` gathered entries: in sh.key / sh.idx when `in_lds`, else at gkey / gidx.  `nz`: this
// thread's corrections so far of the count of non-zero codes.  Several workgroups (`shares`) may rank the same ranking:
// each settles its share of the entries (scattered accesses to six arrays: one workgroup took 21 us over 700 of them), and
// number 0 writes state and record.  What they read of the ranking's state is never written here.
template <bool LC, bool PQ, int THREADS>
__device__ inline void list_rank(const DataArgs& a, const ListArgs& w, ListShared& sh, u32 s, u32 want, u32 n, bool in_lds, int nz,
                                 u32 share, u32 shares, condensa_select* results, int n_groups) {
    const u32 tid = threadIdx.x;
    Slot& slot = a.slots[s];
    const u32 g = s / a.J, j = s - g * a.J;
    condensa_select* record = results + static_cast<u64>(j) * n_groups + g;
    const u32 want_all = want;
    const bool nothing = slot.k == 0;                      // nothing is kept, and the sweep kept nothing
    if (nothing) {
        if (tid == 0 && share == 0) *record = select_record(slot, false, 0, 0, 0, 0, slot.path);
    } else if (want != 0) {                                // 0: it failed
        const u32* __restrict__ gkey = w.gkey + static_cast<u64>(s) * w.gather_cap;
        const u32* __restrict__ gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
        if (!in_lds && n <= kListRanked) {
            for (u32 i = tid; i < n; i += THREADS) { sh.key[i] = gkey[i]; sh.idx[i] = gidx[i]; }
            in_lds = true;
        }
        auto key_of = [&](u32 i) { return in_lds ? sh.key[i] : gkey[i]; };
        auto idx_of = [&](u32 i) { return in_lds ? sh.idx[i] : gidx[i]; };
        const ListWin win = w.win[s];
        const u32 bits = win.bins & 0xFFu;                 // low bits of key - lo that the window's bins leave open
        const u32 sub = bits > 8 ? bits - 8 : 0;
        const u32 mask = (1u << (bits - sub)) - 1u;        // at most eight bits
        if (tid < static_cast<u32>(kListBins)) sh.hist[tid] = 0;
        if (tid == 0) sh.r = 0;
        __syncthreads();
        for (u32 i = tid; i < n; i += THREADS) atomicAdd(&sh.hist[((key_of(i) - win.lo) >> sub) & mask], 1u);
        __syncthreads();
        u32 bin, in_bin;
        list_pick(sh, true, want, &bin, &want, &in_bin);
        if (in_bin <= kListPairs) {                        // uniform
            for (u32 i = tid; i < n; i += THREADS) {
                const u32 key = key_of(i);
                if ((((key - win.lo) >> sub) & mask) == bin) {
                    const u32 p = atomicAdd(&sh.r, 1u);
                    sh.pkey[p] = key;
                    sh.pidx[p] = idx_of(i);
                }
            }
            __syncthreads();
            if (tid < in_bin) {
                const u32 key = sh.pkey[tid], idx = sh.pidx[tid];
                u32 higher = 0, same = 0, same_before = 0;
#pragma unroll 8
                for (u32 e = 0; e < in_bin; ++e) {
                    const u32 k2 = sh.pkey[e];
                    higher += k2 > key ? 1u : 0u;
                    same += k2 == key ? 1u : 0u;
                    same_before += (k2 == key && sh.pidx[e] < idx) ? 1u : 0u;
                }
                if (higher + same_before + 1 == want) { sh.T = key; sh.rem = want - higher; sh.n_tie = same; sh.last = idx; }
            }
        } else {
            // many share those bits too (ties above all): radix levels on the whole key, then on the index
            u32 prefix[2] = {0, 0}, rem = want_all, n_eq = 0, b;
            for (int part = 0; part < 2; ++part) {         // 0: key, highest first; 1: index among equal keys, lowest first
                if (part == 1 && tid == 0) { sh.T = prefix[0]; sh.r = rem; sh.n_tie = n_eq; }
                for (int shift = 24; shift >= 0; shift -= 8) {
                    if (tid < static_cast<u32>(kListBins)) sh.hist[tid] = 0;
                    __syncthreads();
                    for (u32 i = tid; i < n; i += THREADS) {
                        const u32 key = key_of(i);
                        if (part == 1 && key != prefix[0]) continue;
                        const u32 v = part == 0 ? key : idx_of(i);
                        if (shift == 24 || (v >> (shift + 8)) == (prefix[part] >> (shift + 8))) atomicAdd(&sh.hist[(v >> shift) & 255u], 1u);
                    }
                    __syncthreads();
                    list_pick(sh, part == 0, rem, &b, &rem, &n_eq);
                    prefix[part] |= b << shift;
                }
            }
            if (tid == 0) { sh.last = prefix[1]; sh.rem = sh.r; }
        }
        __syncthreads();
        const u32 T = sh.T, last = sh.last;
        if (w.write) {
            constexpr int B = 4;
            for (u32 i0 = tid * shares + share; i0 < n; i0 += THREADS * B * shares) {
                u32 idx[B];
                bool keep[B], on[B];
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const u32 i = i0 + b * THREADS * shares;
                    on[b] = i < n;
                    const u32 key = on[b] ? key_of(i) : 0u;
                    idx[b] = on[b] ? idx_of(i) : 0u;
                    keep[b] = key > T || (key == T && idx[b] <= last);
                    on[b] = on[b] && keep[b] != (key >= win.mid);
                }
                list_fix<LC, PQ, B>(a, w, j, idx, keep, on, &nz);
            }
        }
        if (tid == 0 && share == 0) {
            u64 tie_end = slot.n;
            if (sh.rem < sh.n_tie) {
                const TensorDesc& td = a.td[a.chunk_map[last / kChunk]];
                tie_end = static_cast<u64>(last) - td.chunk_start * kChunk + (a.per_tensor ? 0 : td.flat_start) + 1;
            }
            slot.prefix = T; slot.remaining = sh.rem; slot.n_tie = sh.n_tie; slot.need_tie = 0; slot.tie_end = tie_end; slot.state = kDone;
            *record = select_record(slot, true, T, sh.rem, sh.n_tie, tie_end, slot.path);
        }
    }
    if (PQ && w.nnz_out && w.write && (nothing || want_all != 0)) {
        u32 v = static_cast<u32>(nz), total;               // modulo 2^32: the sum itself is smaller
        if (THREADS == kListThreads)                       // alone: the sweep's count, corrected by the passes over the list
            for (u32 i = tid; i < static_cast<u32>(kListSegs); i += THREADS) v += w.nnz[i];
        __syncthreads();
        wg_incl_scan_u32<THREADS>(v, sh.wave, &total);
        if (tid == 0 && THREADS == kListThreads) {
            *w.nnz_out = total;
        } else if (tid == 0) {                             // one of several: corrections of what k_list_gather stored
            const long long d = static_cast<int>(total) + (share == 0 ? static_cast<long long>(a.ctl->nnz_delta) : 0ll);
            if (d != 0) atomicAdd(reinterpret_cast<unsigned long long*>(w.nnz_out), static_cast<unsigned long long>(d));
        }
    }
    __syncthreads();                                       // the shared words are free for the next ranking
}

// Rankings of populations of at most list_lone elements: one workgroup each does the counting, the gathering and the
// ranking on its list, and a failed ranking by itself (it reads the population a few times over: a megabyte or so).
// 22 thousand listed keys of a 1024x1024 matrix: see the measurements beside the launch rule.
template <bool LC, bool PQ>
__global__ __launch_bounds__(kListThreads) void k_list_finish(DataArgs a, ListArgs w, condensa_select* results, int n_groups) {
    constexpr u32 kQueue = 4096;
    __shared__ ListShared sh;
    __shared__ __align__(8) u32 s_big[kQueue];             // queue of wrong decisions; the failed case: a histogram of kBins
    __shared__ u32 s_n, s_f, s_over, s_want, s_bin, s_found;
    __shared__ u64 s_rem, s_cnt;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    constexpr u32 kWaves = kListThreads / 64;
    const u32 s = blockIdx.x;
    const ListRank rk = w.rank[s];
    const ListWin win = w.win[s];
    const u32 g = s / a.J, j = s - g * a.J;
    Slot& slot = a.slots[s];
    int nz = 0;
    u32 want = 0, n = 0;
    bool in_lds = false;
    const bool selecting = slot.state == kSelecting;
    if (selecting) {                                       // uniform
        const u64 cw = tid < rk.n_segs ? w.cnt[static_cast<u64>(s) * w.max_segs + tid] : 0;       // n_segs <= kListSegs == kListThreads
        const u32 k = static_cast<u32>(slot.k);
        if (tid < static_cast<u32>(kListBins)) sh.hist[tid] = 0;
        if (tid == 0) { s_n = 0; s_f = 0; s_over = 0; s_want = 0; }
        __syncthreads();
        if (static_cast<u32>(cw) > rk.seg_cap) s_over = 1;
        u32 kept, listed;
        wg_incl_scan_u32<kListThreads>(static_cast<u32>(cw >> 32), sh.wave, &kept);
        wg_incl_scan_u32<kListThreads>(static_cast<u32>(cw), sh.wave, &listed);
        const u32 lo = win.lo, shift = win.bins & 0xFFu, mid_bin = win.bins >> 8;
        list_walk(w, s, rk, wave, kWaves, [&](bool there, u32 key, u64) {
            if (there) atomicAdd(&sh.hist[(key - lo) >> shift], 1u);
        });
        __syncthreads();
        if (wave == 0) {                                   // listed keys from the estimate on
            u32 gt = 0;
            for (u32 b = lane; b < static_cast<u32>(kListBins); b += 64) gt += b >= mid_bin ? sh.hist[b] : 0u;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) gt += __shfl_xor(gt, d, 64);
            const u32 above = kept - gt;                   // keys above the window
            if (lane == 0 && s_over == 0 && kept >= gt && above < k && k - above <= listed) s_want = k - above;
        }
        __syncthreads();
        want = s_want;
        if (want != 0) {                                   // uniform
            u32 bin;
            list_pick(sh, true, want, &bin, &want, &n);
            if (n > w.gather_cap) want = 0;
            u32* gkey = w.gkey + static_cast<u64>(s) * w.gather_cap;
            u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
            const u32* __restrict__ ids = w.idx + rk.base;
            in_lds = n <= kListRanked;
            if (want != 0) {
                list_walk(w, s, rk, wave, kWaves, [&](bool there, u32 key, u64 at) {
                    const u32 b = (key - lo) >> shift, entry = static_cast<u32>(at - rk.base);
                    const bool found = there && b == bin, wrong = w.write && there && b != bin && (b > bin) != (b >= mid_bin);
                    const u32 f = wave_push(&s_f, found);  // n of them; their indices are fetched below, side by side
                    if (found) {
                        if (in_lds) { sh.key[f] = key; sh.idx[f] = entry; }
                        else        { gkey[f] = key; gidx[f] = entry; }
                    }
                    const u32 q = wave_push(&s_n, wrong);
                    if (wrong) {
                        if (q < kQueue) s_big[q] = entry | (b > bin ? 0x80000000u : 0u);
                        else            list_fix_one<LC, PQ>(a, w, j, ids[entry], b > bin, &nz);
                    }
                });
                __syncthreads();
                if (in_lds) for (u32 f = tid; f < n; f += kListThreads) sh.idx[f] = ids[sh.idx[f]];
                else        for (u32 f = tid; f < n; f += kListThreads) gidx[f] = ids[gidx[f]];
                list_fix_queue<LC, PQ, kListThreads>(a, w, j, ids, s_big, s_n < kQueue ? s_n : kQueue, &nz);
                __threadfence_block();                     // the gathered entries are read by other threads below
                __syncthreads();
            }
        }
    }
    list_rank<LC, PQ, kListThreads>(a, w, sh, s, want, n, in_lds, nz, 0, 1, results, n_groups);
    if (!selecting || want != 0) return;
    // failed: radix levels over the population, the tie rule, and every output again
    const u64 cb = a.per_tensor ? a.td[g].chunk_start : 0, ce = a.per_tensor ? a.td[g + 1].chunk_start : a.n_chunks;
    constexpr int kRun = kChunk / kListThreads;            // consecutive elements per thread
    auto keys_of = [&](u64 c, u32* key) -> int {           // keys of this thread's run of chunk c; how many exist
        const TensorDesc& td = a.td[a.chunk_map[c]];
        const u64 e0 = (c - td.chunk_start) * kChunk + tid * kRun;
        int have = 0;
#pragma unroll
        for (int i = 0; i < kRun; ++i)
            if (e0 + i < td.n) { key[i] = mag_key(LC ? lc_shift(td.w[e0 + i], td.lam[e0 + i], a.mu) : td.w[e0 + i]); have = i + 1; }
        return have;
    };
    u64 rem = slot.k, n_tie = 0;
    u32 T = 0;
    for (int level = 0; level < n_levels(31); ++level) {
        const Level L = level_of(31, level);
        const int nb = 1 << L.bits;
        for (int i = tid; i < kBins; i += kListThreads) s_big[i] = 0;
        if (tid == 0) s_found = 0;
        __syncthreads();
        for (u64 c = cb; c < ce; ++c) {
            u32 key[kRun];
            const int have = keys_of(c, key);
            for (int i = 0; i < have; ++i)
                if (((static_cast<u64>(key[i]) ^ T) >> L.hi_shift) == 0) atomicAdd(&s_big[(key[i] >> L.shift) & (nb - 1)], 1u);
        }
        __syncthreads();
        if (wave == 0) wave_pick_desc(s_big, nb, rem, &s_bin, &s_rem, &s_cnt, &s_found);
        __syncthreads();
        T |= s_bin << L.shift;
        rem = s_rem;
        n_tie = s_cnt;
        __syncthreads();
    }
    u64 tie_end = slot.n;
    if (rem < n_tie) {                                     // uniform: the chunk and the element that end the kept ties
        u64 cum = 0;
        for (u64 c = cb; c < ce; ++c) {
            u32 key[kRun], hits = 0, total;
            const int have = keys_of(c, key);
            for (int i = 0; i < have; ++i) hits += key[i] == T ? 1u : 0u;
            const u32 before = wg_incl_scan_u32<kListThreads>(hits, sh.wave, &total) - hits;
            if (cum + total >= rem) {                      // uniform
                u64 seen = cum + before;
                const TensorDesc& td = a.td[a.chunk_map[c]];
                for (int i = 0; i < have; ++i)
                    if (key[i] == T && ++seen == rem) s_rem = (c - td.chunk_start) * kChunk + tid * kRun + i + (a.per_tensor ? 0 : td.flat_start) + 1;
                break;
            }
            cum += total;
        }
        __syncthreads();
        tie_end = s_rem;
    }
    u32 codes = 0;
    if (w.write)
        for (u64 c = cb; c < ce; ++c) {
            u32 key[kRun];
            const int have = keys_of(c, key);
            const TensorDesc& td = a.td[a.chunk_map[c]];
            const u64 e0 = (c - td.chunk_start) * kChunk + tid * kRun, flat = e0 + (a.per_tensor ? 0 : td.flat_start);
            for (int i = 0; i < have; ++i) {
                const bool keep = keep_rule(key[i], T, flat + i, tie_end);
                int dummy = 0;
                list_fix_one<LC, PQ>(a, w, j, static_cast<u32>(c) * kChunk + tid * kRun + i, keep, &dummy);
                if (PQ && keep && (f32_to_f16_rne(lc_shift(td.w[e0 + i], td.lam[e0 + i], a.mu)) & 0x7FFFu) != 0) ++codes;
            }
        }
    __syncthreads();
    if (PQ && w.nnz_out && w.write) {
        u32 total;
        wg_incl_scan_u32<kListThreads>(codes, sh.wave, &total);
        if (tid == 0) *w.nnz_out = total;
    }
    if (tid == 0) {
        slot.prefix = T; slot.remaining = rem; slot.n_tie = n_tie; slot.need_tie = 0; slot.tie_end = tie_end; slot.state = kDone;
        results[static_cast<u64>(j) * n_groups + g] = select_record(slot, true, T, rem, n_tie, tie_end, 3);
    }
}

// The failed case: ranks the populations that the windows did not resolve by three radix levels over the weights, then applies every
// result again: one phase for the
// others, 5 phases per failed ranking and one or two at the end, each cut into gridDim.x pieces.  The pieces are
// handed out in order by a ticket counter, and a piece of phase p first waits until every piece of the phases before
// it is done.  All of those were handed out earlier, to workgroups that are running or have ended, and the earliest
// unfinished phase waits for nothing, so every wait ends whatever part of the grid the device holds at a time.
// What one phase hands to the next is written and read with device-scope operations.
constexpr int kSettleGrid = 512;

__device__ inline u32 ld_dev(const u32* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void st_dev(u32* p, u32 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The bin (of kBins, walked from the top) that holds descending rank r; all kBlock threads, returns with a barrier.
__device__ inline void fallback_pick(const u32* hist, u64 r, u64* s_wave, u64* s_pick) {
    constexpr int kPer = kBins / kBlock;
    u32 c[kPer];
    u64 sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) { c[i] = ld_dev(hist + kBins - 1 - (threadIdx.x * kPer + i)); sum += c[i]; }
    u64 total;
    u64 before = block_excl_scan_u64(sum, s_wave, &total);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (before < r && r <= before + c[i]) { s_pick[0] = kBins - 1 - (threadIdx.x * kPer + i); s_pick[1] = r - before; s_pick[2] = c[i]; }
        before += c[i];
    }
    __syncthreads();
}

template <bool LC, bool VEC, bool PQ>
__global__ __launch_bounds__(kBlock) void k_list_settle(DataArgs a, ListArgs w, condensa_select* results, int n_groups, int vec_out) {
    __shared__ u32 s_hist[kBins];
    __shared__ u64 s_wave[kBlock / 64], s_pick[3], s_at[3];
    __shared__ u32 s_ticket;
    __shared__ ListShared s_rank;
    const u32 n_fail = w.fb->failed;                       // final: an earlier kernel counted
    if (n_fail == 0) {
        const u32 n_r = static_cast<u32>(w.n_rankings), shares = n_r * 16 <= gridDim.x ? 16u : (n_r <= gridDim.x ? gridDim.x / n_r : 1u);
        for (u32 v = blockIdx.x; v < n_r * shares; v += gridDim.x)
            list_rank<LC, PQ, kBlock>(a, w, s_rank, v / shares, w.bin_want[v / shares], w.gathered[v / shares], false, 0, v % shares, shares, results, n_groups);
        return;
    }
    const int tid = threadIdx.x;
    const u32 G = gridDim.x;
    const bool nnz = PQ && w.write && w.nnz_out != nullptr;
    const u32 rank_phases = 1 + 5 * n_fail;               // phase 0: the rankings that did not fail
    const u32 phases = rank_phases + (w.write ? 1 : 0) + (nnz ? 1 : 0);
    for (;;) {
        __syncthreads();
        if (tid == 0) {
            const u32 ticket = __hip_atomic_fetch_add(&w.fb->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const u32 phase = ticket / G;
            if (phase < phases)
                while (ld_dev(&w.fb->done) < phase * G) __builtin_amdgcn_s_sleep(8);
            s_ticket = ticket;
        }
        __syncthreads();
        __threadfence();                                   // nothing read below may come from before the wait
        const u32 phase = s_ticket / G, piece = s_ticket % G;
        if (phase >= phases) return;                       // every workgroup gets here: tickets only grow
        if (phase == 0) {
            for (u32 s = piece; s < static_cast<u32>(w.n_rankings); s += G) list_rank<LC, PQ, kBlock>(a, w, s_rank, s, w.bin_want[s], w.gathered[s], false, 0, 0, 1, results, n_groups);
        } else if (phase < rank_phases) {
            const u32 f = (phase - 1) / 5, step = (phase - 1) % 5;
            const u32 r = w.fail_list[f];
            const u32 g = r / a.J, j = r % a.J;
            const u64 k = a.slots[r].k;
            u32* hist = w.fb_hist + static_cast<u64>(f & 1) * 3 * kBins;
            const u64 cb = a.per_tensor ? a.td[g].chunk_start : 0, ce = a.per_tensor ? a.td[g + 1].chunk_start : a.n_chunks;
            // digits decided by the levels before this step
            u32 prefix = 0;
            u64 rem = k, n_tie = 0;
            const u32 decided = step < 3 ? step : 3;
            for (u32 l = 0; l < decided; ++l) {
                fallback_pick(hist + l * kBins, rem, s_wave, s_pick);
                prefix |= static_cast<u32>(s_pick[0]) << level_of(31, l).shift;
                rem = s_pick[1];
                n_tie = s_pick[2];
                __syncthreads();
            }
            if (step < 3) {
                const Level L = level_of(31, step);
                const int nb = 1 << L.bits;
                for (int i = tid; i < kBins; i += kBlock) s_hist[i] = 0;
                __syncthreads();
                for (u64 c = cb + piece; c < ce; c += G) {
                    const TensorDesc& td = a.td[a.chunk_map[c]];
                    const u64 base = (c - td.chunk_start) * kChunk;
                    for (int q = 0; q < kQuadsPerThread; ++q) {
                        const u64 e0 = base + static_cast<u64>(q) * (kBlock * 4) + tid * 4;
                        if (e0 >= td.n) break;
                        float v[4], l[4];
                        load4<VEC>(td.w, e0, td.n, v);
                        if (LC) load4<VEC>(td.lam, e0, td.n, l);
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            if (e0 + x >= td.n) break;
                            const u32 key = mag_key(LC ? lc_shift(v[x], l[x], a.mu) : v[x]);
                            if (((static_cast<u64>(key) ^ prefix) >> L.hi_shift) == 0) atomicAdd(&s_hist[(key >> L.shift) & (nb - 1)], 1u);
                        }
                    }
                }
                __syncthreads();
                for (int i = tid; i < nb; i += kBlock)
                    if (s_hist[i]) __hip_atomic_fetch_add(&hist[step * kBins + i], s_hist[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else if (step == 3) {
                // ties per chunk; piece 0 also clears the other set of histograms, whose ranking is finished
                if (piece == 0)
                    for (int i = tid; i < 3 * kBins; i += kBlock) st_dev(w.fb_hist + static_cast<u64>((f + 1) & 1) * 3 * kBins + i, 0u);
                for (u64 c = cb + piece; c < ce; c += G) {
                    const TensorDesc& td = a.td[a.chunk_map[c]];
                    const u64 base = (c - td.chunk_start) * kChunk;
                    u64 mine = 0;
                    for (int q = 0; q < kQuadsPerThread; ++q) {
                        const u64 e0 = base + static_cast<u64>(q) * (kBlock * 4) + tid * 4;
                        if (e0 >= td.n) break;
                        float v[4], l[4];
                        load4<VEC>(td.w, e0, td.n, v);
                        if (LC) load4<VEC>(td.lam, e0, td.n, l);
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            if (e0 + x >= td.n) break;
                            mine += mag_key(LC ? lc_shift(v[x], l[x], a.mu) : v[x]) == prefix ? 1u : 0u;
                        }
                    }
                    u64 total;
                    block_excl_scan_u64(mine, s_wave, &total);
                    if (tid == 0) st_dev(&a.tiecnt[c], static_cast<u32>(total));
                }
            } else if (piece == 0) {
                // the index that ends the kept ties, then state and record
                u64 tie_end = a.slots[r].n;
                if (rem < n_tie) {                         // uniform
                    if (tid == 0) s_at[2] = 0;
                    u64 cum = 0;
                    for (u64 c0 = cb; c0 < ce; c0 += kBlock) {           // uniform trip count
                        const u64 c = c0 + tid;
                        const u64 x = c < ce ? ld_dev(&a.tiecnt[c]) : 0;
                        u64 total;
                        const u64 ex = cum + block_excl_scan_u64(x, s_wave, &total);
                        if (ex < rem && rem <= ex + x) { s_at[0] = c; s_at[1] = rem - ex; s_at[2] = 1; }
                        cum += total;
                    }
                    __syncthreads();
                    if (s_at[2]) {
                        const u64 c = s_at[0], want = s_at[1];
                        const TensorDesc& td = a.td[a.chunk_map[c]];
                        constexpr int kRun = kChunk / kBlock;            // consecutive elements per thread
                        const u64 e0 = (c - td.chunk_start) * kChunk + static_cast<u64>(tid) * kRun;
                        u32 eq = 0;
                        for (int x = 0; x < kRun; ++x)
                            if (e0 + x < td.n && mag_key(LC ? lc_shift(td.w[e0 + x], td.lam[e0 + x], a.mu) : td.w[e0 + x]) == prefix) eq |= 1u << x;
                        u64 total;
                        const u64 before = block_excl_scan_u64(__popc(eq), s_wave, &total);
                        if (before < want && want <= before + __popc(eq)) {
                            for (u64 skip = want - before - 1; skip > 0; --skip) eq &= eq - 1;
                            s_at[0] = (a.per_tensor ? 0 : td.flat_start) + e0 + (__ffs(eq) - 1) + 1;
                        }
                        __syncthreads();
                        tie_end = s_at[0];
                    }
                }
                if (tid == 0) {
                    Slot& slot = a.slots[r];
                    slot.prefix = prefix; slot.remaining = rem; slot.n_tie = n_tie; slot.need_tie = 0; slot.tie_end = tie_end;
                    slot.state = kDone;
                    results[static_cast<u64>(j) * n_groups + g] = select_record(slot, true, prefix, rem, n_tie, tie_end, 3);
                }
            }
        } else if (w.write && phase == rank_phases) {
            if (LC) {
                constexpr u32 kPer = kChunk / (kBlock * 4);
                for (u64 tile = piece; tile < a.n_chunks * kPer; tile += G) {
                    if (VEC && vec_out) lc_apply_tile<true, kBlock, PQ, 1>(a, w.out, tile);
                    else                lc_apply_tile<false, kBlock, PQ, 1>(a, w.out, tile);
                }
            } else {
                for (u64 tile = piece; tile < a.n_chunks * kSubPerChunk; tile += G) {
                    if (VEC && vec_out) prune_apply_tile<true>(a, w.out, tile);
                    else                prune_apply_tile<false>(a, w.out, tile);
                    __syncthreads();                       // the tile's LDS tables are rewritten by the next one
                }
            }
        } else if (piece == 0) {
            u64 v = 0, total;
            for (int i = tid; i < kNnzSegs; i += kBlock)
                v += __hip_atomic_load(&a.nnz_seg[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            block_excl_scan_u64(v, s_wave, &total);
            if (tid == 0) *w.nnz_out = total;
        }
        __threadfence();                                   // every thread's stores reach the device before the piece counts as done
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_add(&w.fb->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace condensa
