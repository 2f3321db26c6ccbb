// Listed windows: the selection of ordinary calls (the rule is want_list, either scope) in three to seven launches (one ranking: three).
//
// Up to some ten million weights a call is bound by its dependent launches (about 4.5 us each, however little they
// do) and by how often it reads the weights, which the three histogram sweeps of the radix levels make four times.
// Here
//   1. k_begin_sample (or k_begin and k_list_sample): every workgroup ranks its own sample in LDS.  For a ranking it wants
//      the sample keys at the expected rank of the threshold and a little to either side of it.  Small populations get one
//      workgroup, whose bounds lie as many standard deviations of the sample rank apart as the call asks for.  Large ones
//      get up to kListMaxW, each with a sample spread over the whole population, and list_bounds (a workgroup at the end of
//      the same launch, or k_list_bounds) takes mean and deviation of their keys, or order statistics where these look
//      nothing like a normal distribution's: a confidence interval for the threshold that needs no assumption about how
//      neighbours correlate.
//      Either way: a window [lo, hi] that holds the threshold unless the sample was unlucky, and an estimate `mid`.
//   2. k_list_sweep / k_list_sweep_multi: ONE pass over the weights writes the outputs (final outside the windows,
//      provisional -- kept from `mid` on -- inside), counts the keys above each window and lists the keys inside it
//      with their indices.
//   3. The lists are counted in kListBins bins over their windows (several rankings: k_list_hist; one: the sweep itself).
//      k_list_gather finds the bin of rank k - above, settles the listed elements outside it (their outputs are rewritten
//      where the provisional decision was wrong) and gathers those inside, a few hundred.
//   4. k_list_settle ranks these, applies the tie rule, writes state and record and settles them too.  Rankings that the
//      lists leave open (the window missed, or the list overflowed, or thousands of ties) go on from there, all of them
//      together in a few passes over the weights that the whole grid takes (list_fallback).
//      One ranking: 3 and 4 are one launch, k_list_resolve.
// Weights with many equal magnitudes -- pruned before, widened from 8-bit codes -- are such rankings as a rule, so the
// sample also says when a list could not hold its window (kListCrowded): the sweep then leaves that ranking out.
// Microseconds at the threshold density 0.1 to 0.2, radix levels / one ranking after the other, by tickets / now: 20 M
// weights of a VGG-19, nine tenths zeros 409 / 1052 / 146, E4M3 values 180 / 1000 / 136; layer by layer, zeros 365 / 7859 /
// 220, E4M3 values 185 / 4453 / 224; ten densities, E4M3 values 269 / 6941 / 416; 2^18 weights, zeros 680 / 1227 / 62.
// One workgroup draws some 25 GB/s from memory it did not write, so the lists (10^5 entries) are walked by many.  When
// no population exceeds list_lone elements, its list is short enough for one workgroup to do 3 and 4 alone
// (k_list_finish): three launches, and a ranking that it leaves open stays with that workgroup (list_alone).
// Results never depend on the sample.  Section 3.1 (a sparsity turned into a magnitude threshold), Section 3.3 (the
// C step and the multiplier update), Results (up to ten samples per search share a pass).
#pragma once
#include <type_traits>
#include "host.h"
#include "k_apply.h"
#include "k_small.h"
#include "k_window.h"

namespace condensa {

constexpr int kListThreads = 1024;
constexpr int kListSegs = 1024;                  // segments of a ranking's list at most
constexpr int kListMaxW = 256;                   // sampling workgroups of one population at most
constexpr int kListMaxRankings = 4096;
constexpr int kListBins = 256;                   // bins over a window
static_assert(kListBins == 1 << 8, "list_window: 32 - 8 bits");
constexpr u32 kListRanked = 2048;                // gathered entries that are held in LDS
constexpr u32 kListGather = 1u << 18;            // gathered entries of a ranking at most; with more (ties) it is left open
// ... of one GLOBAL ranking whose list is long: as many as values of binary16 have equals there (N / 2100 at the most); left open, they cost two more sweeps (1.2 G
// such weights, 380 thousand ties: L-C step 12 970 -> 3 990 us, pruned 6 550 -> 1 895; such calls' workspaces
// have room for the sampled window, which is more).
constexpr u32 kListGatherLong = 1u << 20;
constexpr u32 kListLine = 32;                    // words of a 128-byte line
// Lists of at least so many elements are long: from there on their bins outgrow kListFound (201 M weights: 4.1 thousand entries at the most), and posting to the
// larger arrays costs up to 8 us: pruning 151 M weights 250 us short and 258 long, 189 M 302 and 309, L-C step 517 and 524, 624 and 630; 208 M 338 either way.
constexpr u64 kListLong = static_cast<u64>(3) << 26;
inline bool list_long(u64 N) { return N >= kListLong; }
constexpr u32 kListFound = 4096;                 // entries of the threshold's bin that k_list_resolve ranks from LDS
constexpr u32 kListPosted = 65536;               // ... and of long lists: 1.2 G weights 12 to 25 thousand as their threshold lies in its binade, more where rows differ in size
constexpr u32 kListRow = 64;                     // segments are multiples of this many entries

// Populations up to here are sampled and finished by one workgroup.  Several densities: the windows of one sampling workgroup
// overlap, and the sweep's general path is slow.  One ranking alone: 2^18 weights take 38-46 us that way (tied ones up to
// 250), 39 with the lists walked by many (tied ones 65-90).  One of many rankings: the workgroups of the others fill the
// chip (96 matrices of 2^18 and 2^20 weights 160 us, 203 with 32 sampling workgroups for each).
inline u64 list_lone(int J, bool per_tensor) { return static_cast<u64>(1) << (J > 1 ? 16 : (per_tensor ? 18 : 17)); }

// Sampling workgroups of a population of n elements: the window is narrowed as the population grows.  One workgroup leaves
// a window of up to 8 % of it (10 sd of its rank); 32 about 1 %, 64 about 0.7 %, 256 about 0.3 %, at the cost of some 3 us (their
// bounds).  Above list_lone that is earned back at once: 295 thousand weights in two densities 52.3 us with one, 37.7 with 32;
// 600 thousand 59.7 and 39.5; pruning 700 thousand in one density 37.3 and 36.5 (when the bounds were a launch of 4.5 us).
inline u32 list_sample_groups(u64 n, int J, bool per_tensor) {
    if (n <= list_lone(J, per_tensor)) return 1;
    if (n <= (static_cast<u64>(1) << 21)) return 32;
    if (n <= (static_cast<u64>(1) << 23)) return 64;
    return kListMaxW;
}
// Sampling workgroups that are resident at once (two to a compute unit, less those that begin the call and bound the windows): what
// goes beyond that waits for another round of 8 us, so PER_TENSOR populations that ask for more get half as many at most, and again,
// down to a quarter of what list_sample_groups says, and 32.
constexpr u32 kSampleResident = 480;
inline u32 list_fewer_groups(u32 asked, u32 most) {
    const u32 least = asked / 4 < 32 ? 32 : asked / 4;
    return asked < most ? asked : (most < least ? (least < asked ? least : asked) : most);
}
// Sample positions per thread: 1 where several workgroups sample, 4 where one does alone.  Also 4 beyond 2^26 elements (in quads): half the window for
// 6 us more.  A window of 256 sampling workgroups of one unit left more than kListFound entries in the threshold's bin of 2^27 weights at
// density 0.6, and the whole grid ranked them (65 us where hist, gather and settle took 52); now 20.  And 4 for populations that got
// fewer workgroups than list_sample_groups says: neighbours resemble each other where rows differ in size, so what narrows a window
// is the number of lines that are read, and the lists are sized for it.  With 1 unit, 16 matrices of 9 M weights whose rows' sizes
// vary (normally distributed logarithms, deviation 0.5) overflowed 8 of their lists: 1065 us the call, now 257; 16 of 2.4 M 268 and 98.
// 2 do for those of up to 2^23 elements where the workspace has room for lists twice as long (4: VGG-19 per layer 3 us more).
constexpr u32 kListUnits = 4;
constexpr u32 kSampleDeep = 1u << 24;
enum : u32 { kFewerNone = 0, kFewerLong = 1, kFewerDeep = 2 };   // which of these: none are fewer, those have longer lists, they have not
__host__ __device__ inline bool list_fewer(u32 W, u64 n) { return W != 1 && ((n > (1u << 23) && W < static_cast<u32>(kListMaxW)) || (n > (1u << 21) && W < 64)); }
__host__ __device__ inline u32 list_units(u32 W, u32 quads, u32 fewer) {
    if (W == 1 || quads > kSampleDeep) return kListUnits;
    if (fewer == kFewerNone || !list_fewer(W, static_cast<u64>(quads) * 4)) return 1;
    return fewer == kFewerLong && quads <= (1u << 21) ? 2 : kListUnits;
}
// Entries of a ranking's list: some four times what its window is expected to hold where weights are independent, every element
// of a tiny one.
__host__ __device__ inline u64 list_capacity(u64 n, int cand_shift) {
    if (cand_shift > 0) return (n >> cand_shift) < 4096 ? 4096 : n >> cand_shift;
    if (n <= 4096) return n;
    const u64 e1 = static_cast<u64>(1) << 18, e2 = static_cast<u64>(1) << 21, e3 = static_cast<u64>(1) << 23;
    const u64 c = n <= e1 ? n / 4 : (n <= e2 ? n / 12 : (n <= e3 ? n / 24 : n / 48));
    const u64 least = n <= e1 ? 4096 : (n <= e2 ? e1 / 4 : (n <= e3 ? e2 / 12 : e3 / 24));
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
// lo = hi = mid = 2^32 - 1: nothing is kept, nothing listed.  kListCrowded: the sample holds so many keys like those at
// the window's ends or its estimate (zeros of a pruned model, values on a grid) that the list could not hold them.  No
// sweep is spent on such a ranking; the fallback takes it from there.
struct ListWin { u32 lo, hi, mid, bins; };       // bins: shift | mid_bin << 8 | kListUneven | kListCrowded
constexpr u32 kListCrowded = 0x80000000u;
// kListUneven: its keys may meet in few bins (list_bounds).
constexpr u32 kListUneven = 0x40000000u;
__host__ __device__ inline u32 win_shift(const ListWin& w) { return w.bins & 0xFFu; }
__host__ __device__ inline u32 win_mid_bin(const ListWin& w) { return (w.bins >> 8) & 0xFFu; }
__host__ __device__ inline bool win_crowded(const ListWin& w) { return (w.bins & kListCrowded) != 0; }
__host__ __device__ inline bool win_uneven(const ListWin& w) { return (w.bins & kListUneven) != 0; }

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
    u32 idle;              // 1: every ranking is crowded
    u32 unused;
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

// What the lists leave open (list_fallback).  Cleared at the start of every call.
constexpr int kFallbackLevels = 6;
struct FallbackCtl {
    u32 special;           // rankings in the list of those that may need it
    u32 ties;              // of these: ties have to be searched (those only suspected are not counted)
    u32 apply;             // of these: outputs have to be written again (the same)
    u32 open[kFallbackLevels + 1];   // rankings whose interval still holds several keys, by level
    u32 unused[6];
};
static_assert(sizeof(FallbackCtl) == 64, "FallbackCtl layout");

struct ListState {         // a ranking that the list did not resolve
    u32 a, b;              // its threshold lies between these, ends included (a == b: it is a)
    u32 rank;              // at this rank from the top
    u32 n;                 // keys there
    u32 flags;
    u32 last;              // when found: last tie kept, as chunk * kChunk + place in the chunk
    u32 unused[2];
};
constexpr u64 kPicked = static_cast<u64>(1) << 63;         // the entry is there
constexpr u32 kRangeKnown = 0x80000000u, kRangeBits = 17;
static_assert(kListPosted < 1u << kRangeBits, "ListArgs::range");
constexpr u64 kWalkerLeft = 1;
constexpr u32 kMaxWalkers = kListSegs / 8;                 // a segment for each of a workgroup's eight wavefronts
constexpr u32 kListParts = 4;                              // wavefronts that share a segment where lists are long
constexpr u32 kStateUnsure = 1;      // the interval is the sample's alone; `rank` counts from the top of the population
constexpr u32 kStateMaybe = 2;       // the gathered entries are many: if all are equal they are the ties, else list_rank takes them
constexpr u32 kStateTied = 4;        // the ties are the gathered entries, and the outputs are right but for theirs

struct ListArgs {
    const ListRank* rank;  // [rankings]
    const u32* group_of;   // PER_TENSOR: [sampling workgroups] tensor each samples
    u64* local;            // [3 J][sampling workgroups] upper bound, lower bound and estimate of a ranking (bit 31: crowded) | tag << 32
    u32 n_local;           // sampling workgroups
    u32 tag;               // of this call's words in `local`
    ListWin* win;          // [rankings]
    ListSorted* sorted;    // [populations], J > 1
    u64* cnt;              // [rankings][max_segs] entries offered | keys above the window << 32
    u32* hist;             // [rankings][hist_copies][kListBins] listed keys by bin of their window
    u32 hist_copies;       // a power of two
    u32 uneven_copies;     // the same for a window whose keys may meet in few bins
    u32 count_in_sweep;    // 1: the sweep counts them (one ranking: two launches less, and its one or two listed keys a wavefront cost it
                           // nothing), 0: k_list_hist (several: 780 thousand updates for ten densities of 20 M weights took 30 us), or
                           // k_list_finish for itself
    u32* arrived;          // one ranking: workgroups that have walked their part of the list << 20 | entries they gathered
    u32* ended;            // one ranking, prune + binary16 step: workgroups that are done
    u64* picked;           // one ranking: [kListFound or kListPosted] gathered entries, index | key << 32 | kPicked
    u32* range;            // one ranking: [kMaxWalkers] where a workgroup's entries stand among these, first | number << kRangeBits | kRangeKnown
    u64* verdict;          // one ranking: [kMaxWalkers] for each workgroup: the last entry kept (as in `picked`), or kWalkerLeft
    u32* gathered;         // [rankings][kListLine] entries in the threshold's bin (a counter in a line of its own)
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
    u32* gmax;             // [rankings] largest gathered key, kept where they are many
    u32* gmaxc;            // [rankings] ... and the complement of the smallest
    FallbackCtl* fb;
    u32* special;          // [rankings] those that list_fallback may have to take
    ListState* state;      // [rankings]
    u32* open_of;          // [populations] bit j: ranking j's interval still holds several keys
    u32* tie_of;           // [populations] bit j: its ties have to be searched
    u32* apply_of;         // [populations] bit j: its outputs have to be written again
    u32* fb_hist;          // [rankings][3][fb_bins]: keys of an interval by bin, and the range of each bin's
    u32* fb_above;         // [rankings] keys above an unsure interval
    u32 fb_bins;           // a power of two
    u32* meet;             // [kMeetWords] where list_fallback's workgroups meet
    int cand_shift;
    const OutDesc* out;
    u64* nnz_out;
    int margin16;
    int write;             // 1: the sweep writes the outputs.  0: selection only, an apply sweep follows
    u32 force;             // kForce...
    u32 fewer;             // kFewer...: populations that have fewer sampling workgroups than they ask for
};

// What workgroups of one launch hand to each other is written and read with device-scope operations.
__device__ inline u32 ld_dev(const u32* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void st_dev(u32* p, u32 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline u32 add_dev(u32* p, u32 v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void max_dev(u32* p, u32 v) { __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline u64 ld_dev64(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void st_dev64(u64* p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void or_dev(u32* p, u32 v) { __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Waits until this wavefront's accesses are done.  The fences emit nothing: they keep the compiler from moving accesses across.
__device__ inline void wait_dev() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "singlethread");
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "singlethread");
}

// ---- sample ------------------------------------------------------------------------------------------

__device__ inline ListWin list_window(u32 hi, u32 lo, u32 mid) {
    ListWin x;
    x.hi = hi;
    x.lo = hi == 0xFFFFFFFFu ? hi : (lo < hi ? lo : hi);
    mid = mid < x.lo ? x.lo : (mid > x.hi ? x.hi : mid);
    const u32 span = x.hi - x.lo;
    const u32 shift = span < static_cast<u32>(kListBins) ? 0u : 24u - static_cast<u32>(__builtin_clz(span));       // span >> shift < kListBins
    const u32 mid_bin = (mid - x.lo) >> shift;
    x.mid = x.lo + (mid_bin << shift);
    x.bins = shift | (mid_bin << 8);
    return x;
}

// From the words of list_sample: upper bound, lower bound, estimate (bit 31: crowded).  marks: kListCrowded, kListUneven.
__device__ inline ListWin list_window_of(const u32* word, bool nothing, u32 marks) {
    if (nothing) return list_window(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
    ListWin x = list_window(word[0] & ~kListCrowded, word[1] & ~kListCrowded, word[2] & ~kListCrowded);
    x.bins |= ((word[0] | word[1] | word[2]) & kListCrowded) | marks;
    return x;
}

// One wavefront, J <= kMaxJ windows (in LDS), `by_rank` kMaxJ + 1 words of LDS.  Lane j places window j; crowded ones are
// left out.
__device__ inline void list_sort(const ListWin* win, int J, u32* by_rank, ListSorted* out) {
    const int lane = threadIdx.x & 63;
    const ListWin mine = lane < J ? win[lane] : ListWin{};
    const bool active = lane < J && mine.hi != 0xFFFFFFFFu && !win_crowded(mine);
    const u32 n = static_cast<u32>(__popcll(__ballot(active)));
    const int n_crowded = __popcll(__ballot(lane < J && win_crowded(mine)));
    u32 p = 0;                                             // windows before this one: higher, or equal and earlier
    const u64 in_order = __ballot(active);
    for (int i = 0; i < J; ++i) {
        const u32 h = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(mine.hi), i));
        if (((in_order >> i) & 1u) && (h > mine.hi || (h == mine.hi && i < lane))) ++p;
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
        out->idle = n_crowded == J ? 1u : 0u;
        out->disjoint = overlap == 0 ? 1u : 0u;
    }
}

// The bin of 256 that holds descending rank r (1 <= r <= all counts together): one wavefront, four bins per lane from
// the top.  The lane that finds it returns true.
__device__ inline bool wave_pick256(const u32* s_hist, u32 r, u32* bin) {
    const u32 lane = threadIdx.x & 63u;
    const uint4 c = *reinterpret_cast<const uint4*>(s_hist + 252 - 4 * lane);
    const u32 sum = c.x + c.y + c.z + c.w, incl = wave_incl_scan_u32(sum);
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
    u32 n, chunk_start;    // (32 bits index the elements of these calls)
};

// One sampling workgroup of a population: number `me` of W, whose results go to place `at_local`.  Bound by latency
// (scattered reads, then a chain of six barriers): 7.9 us from the launch to the words for the one density of 20 M weights and
// for ten, 10.3 and 12.9 when every wanted rank was looked for by every thread, in binary64, with eleven barriers.  A lone workgroup writes the window: the rank rule is that of
// sample_rank.  One of several leaves the keys at its expected rank and two ranks to either side of it (which covers
// the bias of small ranks); list_bounds does the rest.  `first_chunk`, `quads`: the population in chunk space.
// LDS (dynamic): sample_lds.  Two workgroups fit a compute unit.
constexpr int kSampleBits2 = 8, kSampleBins2 = 1 << kSampleBits2;        // 19 of 31 bits: the rest is a twentieth of a percent of the value
// Copies of the first histogram, chosen by lane, so that fewer lanes of a wavefront meet on one counter.
__host__ __device__ inline u32 sample_copies(int J) { return J <= 8 ? 4u : 1u; }
__host__ __device__ inline size_t sample_lds(int J) { return (sample_copies(J) * kBins + kListThreads + 3u * J * kSampleBins2) * sizeof(u32); }

constexpr u32 kSampleNone = 0x7FFFFFFFu;         // a bound without such a rank in the sample
struct SampleShared {
    u64 k[kMaxJ], n[kMaxJ];
    float p[kMaxJ], q[kMaxJ];                    // p = k / n of a ranking, and sqrt(kSampleUnit p (1 - p)) (a sample's ranks are at most 2^14)
    ListWin win[kMaxJ];
    u32 wave[kListThreads / 64];
    u32 want[3 * kMaxJ], bin[3 * kMaxJ], rem[3 * kMaxJ], key[3 * kMaxJ];
};
// UNITS: sample positions (of four keys each) per thread (list_units).  Four lanes take the four float4 of a
// 64-byte line: the traffic of one float4 from each line, for four times the keys (262144 scattered float4 of two arrays took
// 11 us, and the 4096 of one workgroup held up its neighbour on the compute unit for 8).  That neighbours resemble each other
// does not mislead the mean over several workgroups; a lone one's window is ten standard deviations of independent keys to either
// side, and half that of independent float4.
template <bool LC, bool VEC, int UNITS, typename TensorOf, typename RankOf>
__device__ inline void list_sample_units(SampleShared& sh, const ListArgs& w, int J, float mu, u32 W, u32 me, u32 at_local, u64 first_ranking, u32 first_chunk, u32 quads,
                                   TensorOf&& tensor_of, RankOf&& rank_of) {
    extern __shared__ __align__(16) u32 s_dyn[];
    float* const s_p = sh.p;
    float* const s_q = sh.q;
    u64* const s_k = sh.k;
    u64* const s_n = sh.n;
    u32* const s_want = sh.want;
    u32* const s_bin = sh.bin;
    u32* const s_rem = sh.rem;
    u32* const s_key = sh.key;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int R = 3 * J;
    const u32 copies = sample_copies(J);
    u32* const hist0 = s_dyn;                    // [copies][kBins]
    u32* const s_incl = hist0 + copies * kBins;  // [kListThreads] counts up to a thread's bins within its wavefront | those of its first bin << 16
    u32* const hist1 = s_incl + kListThreads;    // [R][kSampleBins2]
    {
        const uint4 z = make_uint4(0, 0, 0, 0);
        for (u32 i = tid; i < copies * kBins / 4; i += kListThreads) reinterpret_cast<uint4*>(hist0)[i] = z;
        for (int i = tid; i < R * kSampleBins2 / 4; i += kListThreads) reinterpret_cast<uint4*>(hist1)[i] = z;
    }
    constexpr int lanes = 4;                     // of a 64-byte line
    const int logu = 31 - __clz(static_cast<int>(UNITS * (kListThreads / lanes) * W));     // a power of two
    const u32 places = (quads + lanes - 1) / lanes;

    // Every lane loads, without a branch (from the last place there is when its own is past the end): a load that only some lanes
    // make is waited for before the next one starts, and four units one after the other took 6 to 10 us.  Tensors of fewer than
    // four elements are left out.
    float v[4 * UNITS], l[LC ? 4 * UNITS : 1];
    u32 valid = 0;
    if (quads != 0) {                            // uniform
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const u32 u = static_cast<u32>((i * kListThreads + tid) / lanes) * W + me;          // below 2^logu: its place is in the u-th of as many stretches
            u32 p = places <= (1u << logu) ? u : static_cast<u32>((static_cast<u64>(u) * places + __umulhi(mix32(u), places)) >> logu);
            p = p * lanes + tid % lanes;
            const bool there = p < quads;
            p = there ? p : quads - 1;
            const u32 c = first_chunk + p / (kChunk / 4);
            const SampleTensor td = tensor_of(c);
            const u32 e0 = (c - td.chunk_start) * kChunk + (p % (kChunk / 4)) * 4;
            const bool whole = td.n >= 4;
            if (there && whole && e0 < td.n) valid |= 0xFu << (4 * i);
            const u32 last = whole ? (td.n - 4) & ~3u : 0u, e = e0 < last ? e0 : last;         // the tail: the four before it
            const float* const wp = whole ? td.w + e : reinterpret_cast<const float*>(w.win);          // (any sixteen bytes)
            const float* const lp = !LC ? nullptr : (whole ? td.lam + e : reinterpret_cast<const float*>(w.win));
            if (VEC) {
                const float4 x = *reinterpret_cast<const float4*>(wp);
                v[4 * i] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
                if (LC) {
                    const float4 y = *reinterpret_cast<const float4*>(lp);
                    l[4 * i] = y.x; l[4 * i + 1] = y.y; l[4 * i + 2] = y.z; l[4 * i + 3] = y.w;
                }
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v[4 * i + k] = wp[k];
                    if (LC) l[4 * i + k] = lp[k];
                }
            }
        }
    }
    if (tid < J) {                               // while the loads are on their way
        u64 k, n;
        rank_of(tid, &k, &n);
        const float p = n ? static_cast<float>(k) / static_cast<float>(n) : 0.0f;
        s_p[tid] = p;
        s_q[tid] = sqrtf(static_cast<float>(kSampleUnit) * p * (1.0f - p));
        s_k[tid] = k;
        s_n[tid] = n;
    }
    __syncthreads();
    constexpr int kShift0 = 20;                  // 11 leading bits of 31
    u32 key[4 * UNITS];
#pragma unroll
    for (int i = 0; i < 4 * UNITS; ++i) {
        key[i] = mag_key(LC ? lc_shift(v[i], l[LC ? i : 0], mu) : v[i]);
        if (valid & (1u << i)) atomicAdd(&hist0[(lane & (copies - 1)) * kBins + (key[i] >> kShift0)], 1u);
    }
    __syncthreads();
    {
        const int b0 = kBins - 1 - 2 * tid, b1 = b0 - 1;                 // bins from the top, two per thread
        u32 c0 = hist0[b0], c1 = hist0[b1];
        for (u32 q = 1; q < copies; ++q) { c0 += hist0[q * kBins + b0]; c1 += hist0[q * kBins + b1]; }
        const u32 incl = wave_incl_scan_u32(c0 + c1);                    // a workgroup has at most 2^14 keys
        s_incl[tid] = incl | (c0 << 16);
        if (lane == 63) sh.wave[wave] = incl;
    }
    __syncthreads();
    // The three ranks of every ranking, a wavefront each: the thread whose bins hold it, then the bin.  From here on a word of
    // hist0 says which ranking's histogram of the next digits its bin has: rankings that meet in a bin share that of the first.
    constexpr u32 kHasBins2 = 0x80000000u;
    u32 S;
    {
        const u32 of_wave = lane < kListThreads / 64 ? sh.wave[lane] : 0u, upto = wave_incl_scan_u32(of_wave);
        S = __shfl(upto, 63, 64);
        for (int r = wave; r < R; r += kListThreads / 64) {
            const int j = r / 3, which = r % 3;  // upper bound, lower bound, estimate
            u32 want = 0;                        // 0: no such rank in the sample, unbounded
            if (s_k[j] != 0 && S != 0) {
                const float all = static_cast<float>(S), ks = s_p[j] * all;
                const float m = (W == 1 ? static_cast<float>(w.margin16) / 16.0f * s_q[j] * sqrtf(all) : 0.0f) + 2.0f;
                float x = which == 0 ? floorf(ks - m) : (which == 1 ? ceilf(ks + m) + 1.0f : floorf(ks + 0.5f));
                if (which == 2) x = x < 1.0f ? 1.0f : (x > all ? all : x);
                if (x >= 1.0f && x <= all) want = static_cast<u32>(x);
            }
            if (lane == 0) s_want[r] = want;
            if (want == 0) continue;             // uniform
            const int in_wave = __ffsll(static_cast<long long>(__ballot(upto >= want))) - 1;
            const u32 before_wave = __shfl(upto - of_wave, in_wave, 64);
            const u32 x = s_incl[in_wave * 64 + lane], incl = before_wave + (x & 0xFFFFu);
            const int in_lane = __ffsll(static_cast<long long>(__ballot(incl >= want))) - 1;
            const u32 up = __shfl_up(incl, 1, 64), prev = lane ? up : before_wave;
            if (lane == in_lane) {
                const u32 b0 = kBins - 1 - 2 * (in_wave * 64 + lane), c0 = x >> 16;
                const bool first = want <= prev + c0;
                const u32 bin = first ? b0 : b0 - 1;
                s_bin[r] = bin;
                s_rem[r] = first ? want - prev : want - prev - c0;
                atomicMax(&hist0[bin], kHasBins2 | (63u - static_cast<u32>(r)));
            }
        }
    }
    __syncthreads();
    constexpr int kShift2 = kShift0 - kSampleBits2;
#pragma unroll
    for (int i = 0; i < 4 * UNITS; ++i) {
        if (!(valid & (1u << i))) continue;
        const u32 h = hist0[key[i] >> kShift0];
        if (h & kHasBins2) atomicAdd(&hist1[(63u - (h & 63u)) * kSampleBins2 + ((key[i] >> kShift2) & (kSampleBins2 - 1))], 1u);
    }
    __syncthreads();
    for (int r = wave; r < R; r += kListThreads / 64) {
        const int j = r / 3, which = r % 3;
        u32 bin = 0, word = kSampleNone;
        bool mine = lane == 0;
        if (s_want[r] != 0) {                    // uniform
            const u32* hist = hist1 + (63u - (hist0[s_bin[r]] & 63u)) * kSampleBins2;
            mine = wave_pick256(hist, s_rem[r], &bin);                   // one lane
            if (mine) {
                const u32 key0 = (s_bin[r] << kShift0) | (bin << kShift2), low = (1u << kShift2) - 1u;
                word = which == 0 ? key0 | low : (which == 1 ? key0 : key0 | ((low + 1u) >> 1));
                // sample keys that share 19 bits with this one
                if (static_cast<u64>(hist[bin]) * s_n[j] > list_capacity(s_n[j], w.cand_shift) * S) word |= kListCrowded;
            }
        }
        if (!mine) continue;
        if (W == 1) s_key[r] = which != 0 && word == kSampleNone ? 0u : word;
        else        st_dev64(&w.local[static_cast<u64>(r) * w.n_local + at_local], (static_cast<u64>(w.tag) << 32) | word);
    }
    if (W != 1) return;                          // uniform
    __syncthreads();
    if (tid < J) {
        const ListWin x = list_window_of(s_key + 3 * tid, s_k[tid] == 0, 0u);
        w.win[first_ranking + tid] = x;
        sh.win[tid] = x;
    }
    if (J > 1) {
        __syncthreads();
        if (wave == 0) list_sort(sh.win, J, s_want, w.sorted + first_ranking / J);
    }
}

template <bool LC, bool VEC, typename TensorOf, typename RankOf>
__device__ inline void list_sample(const ListArgs& w, int J, float mu, u32 W, u32 me, u32 at_local, u64 first_ranking, u32 first_chunk, u32 quads,
                                   TensorOf&& tensor_of, RankOf&& rank_of) {
    __shared__ SampleShared sh;
    const u32 units = list_units(W, quads, w.fewer);
    if (units == kListUnits) list_sample_units<LC, VEC, kListUnits>(sh, w, J, mu, W, me, at_local, first_ranking, first_chunk, quads, tensor_of, rank_of);
    else if (units == 2)     list_sample_units<LC, VEC, 2>(sh, w, J, mu, W, me, at_local, first_ranking, first_chunk, quads, tensor_of, rank_of);
    else                     list_sample_units<LC, VEC, 1>(sh, w, J, mu, W, me, at_local, first_ranking, first_chunk, quads, tensor_of, rank_of);
}

// The sampling workgroups as a launch of their own.
template <bool LC, bool VEC>
__global__ __launch_bounds__(kListThreads, 8) void k_list_sample(DataArgs a, ListArgs w) {
    const u32 g = a.per_tensor ? w.group_of[blockIdx.x] : 0u;
    const u64 r0 = static_cast<u64>(g) * a.J;
    const ListRank rk = w.rank[r0];
    const TensorDesc& tg = a.td[a.per_tensor ? g : 0];
    list_sample<LC, VEC>(w, a.J, a.mu, rk.n_groups, blockIdx.x - rk.group0, blockIdx.x, r0, a.per_tensor ? static_cast<u32>(tg.chunk_start) : 0u,
                         static_cast<u32>(a.per_tensor ? (tg.n + 3) / 4 : a.n_chunks * (kChunk / 4)),
                         [&](u32 c) {
                             const TensorDesc& td = a.per_tensor ? tg : a.td[a.chunk_map[c]];
                             return SampleTensor{td.w, td.lam, static_cast<u32>(td.n), static_cast<u32>(td.chunk_start)};
                         },
                         [&](int j, u64* k, u64* n) { *k = a.slots[r0 + j].k; *n = a.slots[r0 + j].n; });
}

// The sample as part of the launch that begins the call (few tensors): what the sampling workgroups need
// of the tables comes as kernel arguments, so they need not wait for the upload.  One launch less: 4 us.  26 bytes a tensor: the
// argument budget would hold 117 next to the other fields, 96 leaves room for more of these.  Calls of more tensors pay the launch.
constexpr int kBeginSampleTensors = 96;
struct BeginSampleArgs {
    UploadArgs up;
    uint4* zero;
    u64 n_zero;            // 16-byte words
    u32* chunk_map;
    u32 n_chunks;
    int n_tensors;
    u32 groups;            // sampling workgroups: after the one that fetches the tables
    u32 fillers;           // workgroups that clear and write the map: after these.  Then one for each population's bounds
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
// Populations with several sampling workgroups, one workgroup here for each, a wavefront a ranking.  The workgroups' keys at
// the expected rank are as many independent draws around the threshold: their mean estimates it, and the window ends as many
// standard errors of that mean to either side as the call asks for (a few more when the deviation itself is estimated from few
// draws).  That holds for draws from something like a normal distribution.  Where they are not -- a model close to its compressed
// form, whose threshold lies at a gap; weights on a grid; workgroups without such a rank in their sample -- the mean can lie where
// no keys are, the interval can end before them, or a few draws far off stretch it.  So the share of the draws beyond either end
// has to be what it is in a normal distribution, give or take three of its deviations (and not nothing).  Long lists (LONG; elsewhere a wrong decision more costs less than the test): so has the share above the mean.
// Where rows differ in size, a workgroup with many large ones has more keys around the threshold too, and the mean lies 2 to 3 of its deviations too low; the median
// does not (1.2 G such weights, a million wrong decisions less: L-C step 4 104 -> 3 850 us, pruned 1 827 -> 1 775; 604 M 2 033 -> 1 950).  Else order
// statistics W/2 -+ z sqrt(W)/2, which assume nothing, take its place.  Elsewhere they would leave windows 1.3 times as wide for 256
// workgroups and twice for 32, estimates off by 1.25 times as much, and take 1.8 us to find.
// L-C step of VGG-19 whose kept weights stand apart from the others, at their share: 262 us by the mean alone, 103 so.
// Workgroups whose sample is empty (all of its places are tensors too short to be sampled) have no part in either.
// WAIT: the sampling workgroups belong to the same launch.  They come before this one in the grid and wait for nobody; their
// words are there when they carry the call's tag (a word left by something else that looks the same would only misplace the
// window).  In a launch of its own this took 4.9 us and 11 for ten densities.  The wait is bounded: where several such launches share
// the chip, the workgroups that wait may hold the places that others' sampling workgroups need.  Who gives up leaves the ranking to
// list_fallback, as a crowded one.
constexpr int kBoundsThreads = 64 * kMaxJ;
constexpr u32 kBoundsPolls = 8192;               // some 10 ms: longer than what this library's other kernels hold the chip for
__device__ inline float wave_sum_f32(float v) {            // in every lane
    auto add = [](float x, u32 from) { return x + __uint_as_float(from); };
    v = add(v, dpp_or_zero<0x111, 0xF>(__float_as_uint(v)));
    v = add(v, dpp_or_zero<0x112, 0xF>(__float_as_uint(v)));
    v = add(v, dpp_or_zero<0x114, 0xF>(__float_as_uint(v)));
    v = add(v, dpp_or_zero<0x118, 0xF>(__float_as_uint(v)));
    v = add(v, dpp_or_zero<0x142, 0xA>(__float_as_uint(v)));
    v = add(v, dpp_or_zero<0x143, 0xC>(__float_as_uint(v)));
    return __uint_as_float(static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(__float_as_uint(v)), 63)));
}
// LOW: the lowest bits of the words, which say nothing (list_sample: twelve).
template <bool WAIT, bool LONG, u32 LOW = 0xFFFu, typename NothingOf>
__device__ inline void list_bounds(const ListArgs& w, int J, u64 r0, u32 group0, u32 W, NothingOf&& nothing_of) {
    __shared__ ListWin s_win[kMaxJ];
    __shared__ u32 s_order[kMaxJ + 1];
    const int lane = threadIdx.x & 63, j = threadIdx.x >> 6;
    if (j < J) {
        constexpr int kPer = kListMaxW / 64;
        u32 v[3][kPer];                          // upper bound, lower bound, estimate
        // what does not depend on the words: shares of the draws that may lie beyond an end
        const float z = static_cast<float>(w.margin16) / 16.0f, all = static_cast<float>(W), due = 0.5f * erfcf(z * (1.0f + 8.0f / all) * rsqrtf(2.0f * all));
        const float tolerance = 3.0f * sqrtf(due * (1.0f - due) / all);
        const float least_beyond = due - tolerance > 0.0f ? due - tolerance : (due * all >= 3.0f ? 1.0f / all : 0.0f), most_beyond = due + tolerance;
        bool given_up = WAIT && (w.force & kForceNoSample);
        // What is executed once is bound by fetching its instructions, so it is executed once before the words are there (all zero).
        u32 dry = WAIT ? 1 : 0;
        asm volatile("" : "+s"(dry));            // (the compiler would take the loop apart)
        for (;; --dry) {                         // uniform
        if (dry != 0 || given_up) {
#pragma unroll
            for (int q = 0; q < 3 * kPer; ++q) v[q / kPer][q % kPer] = 0;
        }
        for (u32 polls = 0; dry == 0 && !given_up; ++polls) {            // uniform
            bool there = true;
            u64 x[3][kPer];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int q = 0; q < kPer; ++q)
                    x[i][q] = 64u * q + lane < W ? ld_dev64(w.local + static_cast<u64>(3 * j + i) * w.n_local + group0 + 64 * q + lane) : 0;
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    there = there && (64u * q + lane >= W || static_cast<u32>(x[i][q] >> 32) == w.tag);
                    v[i][q] = static_cast<u32>(x[i][q]);
                }
            if (!WAIT || __all(there)) break;
            given_up = polls == kBoundsPolls;
            __builtin_amdgcn_s_sleep(1);
        }
        bool drew[kPer];                         // this lane's workgroups whose sample holds anything
        u32 n_drew = 0, ref = 0;                 // uniform
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            drew[q] = 64u * q + lane < W && (v[2][q] & ~kListCrowded) != kSampleNone;
            const u64 m = __ballot(drew[q]);
            if (n_drew == 0 && m != 0) ref = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(v[2][q]), __ffsll(static_cast<long long>(m)) - 1)) & ~kListCrowded;
            n_drew += static_cast<u32>(__popcll(m));
        }
        u32 word[3], marks = 0, says = 0;        // says: how many say crowded, ten bits for each word
        bool none = false;                       // a workgroup without such a rank in its sample
        float mean[3], sq = 0.0f;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            float sum = 0.0f;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                if (64u * q >= W) break;         // uniform
                const u32 key = v[i][q] & ~kListCrowded;
                says += (v[i][q] >> 31) << (10 * i);
                none = none || (drew[q] && key == kSampleNone);
                const float d = drew[q] ? static_cast<float>(static_cast<int>(key - ref)) : 0.0f;
                sum += d;
                if (i == 2) sq += d * d;
            }
            mean[i] = wave_sum_f32(sum) / static_cast<float>(n_drew);
        }
        says = wave_sum_u32(says);
#pragma unroll
        for (int i = 0; i < 3; ++i) if (2 * ((says >> (10 * i)) & 1023u) > n_drew) marks = kListCrowded;      // most of the workgroups say so
        const bool open = __any(none);
        const float n = static_cast<float>(n_drew), var = (wave_sum_f32(sq) - n * mean[2] * mean[2]) / (n - 1.0f);
        const float off = z * (1.0f + 8.0f / n) * sqrtf(var > 0.0f ? var / n : 0.0f);
        // draws of the estimate beyond the interval's ends, above | below << 10, and << 20 the equal ones among 49 pairs of every 16
        u32 beyond = 0;
        if (drew[0])
            beyond = (dpp_or_zero<0x111, 0xF>(v[2][0]) == v[2][0] ? 1u << 20 : 0u) + (dpp_or_zero<0x112, 0xF>(v[2][0]) == v[2][0] ? 1u << 20 : 0u) +
                     (dpp_or_zero<0x114, 0xF>(v[2][0]) == v[2][0] ? 1u << 20 : 0u) + (dpp_or_zero<0x118, 0xF>(v[2][0]) == v[2][0] ? 1u << 20 : 0u);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            if (64u * q >= W) break;             // uniform
            const float d = static_cast<float>(static_cast<int>((v[2][q] & ~kListCrowded) - ref)) - mean[2];
            beyond += drew[q] ? (d > off ? 1u : 0u) + (d < -off ? 0x400u : 0u) : 0u;
        }
        beyond = wave_sum_u32(beyond);
        const u32 above = beyond & 0x3FFu, below = (beyond >> 10) & 0x3FFu, equal = beyond >> 20;
        const u32 fewer = above < below ? above : below, more = above < below ? below : above;
        const bool even = static_cast<float>(fewer) >= n * least_beyond && static_cast<float>(more) <= n * most_beyond;
        bool skewed = false;
        if constexpr (LONG) {
            u32 over = 0;                        // above their mean
#pragma unroll
            for (int q = 0; q < kPer; ++q) over += static_cast<u32>(__popcll(__ballot(drew[q] && static_cast<float>(static_cast<int>((v[2][q] & ~kListCrowded) - ref)) > mean[2])));
            skewed = fabsf(static_cast<float>(over) - 0.5f * n) > 0.75f * sqrtf(n);                  // 2.5 deviations of what it is in a normal distribution
        }
        const bool alike = open || !even || equal >= (W < 64 ? 5u : 9u);         // the last: weights on a grid (3 are equal where they are not)
        if (alike) marks |= kListUneven;
        const bool all_equal = !(var > 0.0f);
        if (!open && ((even && !skewed) || all_equal)) {
            auto at = [&](float d) {             // a key; ref + d may lie outside
                const float least = -static_cast<float>(ref), most = static_cast<float>(0x7FFFFFFFu - ref);
                return d <= least ? 0u : (d >= most ? 0x7FFFFFFFu : ref + static_cast<u32>(static_cast<int>(d)));
            };
            const u32 half = (LOW + 1u) / 2;
            const u32 hi = at(mean[0] + off), lo = at(mean[1] - off);
            word[0] = hi < 0x7FFFFFFFu - half ? hi + half : 0x7FFFFFFFu;
            word[1] = lo < half ? 0u : lo - half;
            word[2] = at(mean[2]);
        } else {
            const u32 h = n_drew / 2, d = static_cast<u32>(fminf(ceilf(z * 0.5f * sqrtf(n)), static_cast<float>(h)));
            const u32 pick[3] = {h + d < n_drew ? h + d : n_drew - 1, h > d ? h - 1 - d : 0u, h};
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                word[i] = 0;
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    v[i][q] &= ~kListCrowded;
                    if (i == 1 && v[i][q] == kSampleNone) v[i][q] = 0;
                    if (!drew[q]) v[i][q] = 0xFFFFFFFFu;
                }
            }
            for (u32 bit = 0x40000000u; bit > LOW; bit >>= 1)         // the largest keys with at most that many of them below
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    u32 n_below = 0;
#pragma unroll
                    for (int q = 0; q < kPer; ++q) n_below += static_cast<u32>(__popcll(__ballot(v[i][q] < (word[i] | bit))));
                    if (n_below <= pick[i]) word[i] |= bit;
                }
            word[0] |= LOW;
            word[2] |= (LOW + 1u) / 2;
        }
        if (given_up || n_drew < 2) { word[0] = 0x7FFFFFFFu; word[1] = 0; marks = kListCrowded; }
        const ListWin x = list_window_of(word, nothing_of(j), marks);
        if (dry != 0) continue;
        if (lane == 0) {
            s_win[j] = x;
            w.win[r0 + j] = x;
        }
        break;
        }
    }
    if (J == 1) return;
    __syncthreads();
    if (threadIdx.x < 64) list_sort(s_win, J, s_order, w.sorted + r0 / J);
}

__global__ __launch_bounds__(kBoundsThreads) void k_list_bounds(DataArgs a, ListArgs w) {
    const u64 r0 = static_cast<u64>(blockIdx.x) * a.J;
    const ListRank rk = w.rank[r0];
    if (rk.n_groups == 1) return;                // its windows are written
    auto nothing_of = [&](u32 j) { return a.slots[r0 + j].k == 0; };
    if (w.gather_cap > kListGather) list_bounds<false, true>(w, a.J, r0, rk.group0, rk.n_groups, nothing_of);       // uniform
    else                            list_bounds<false, false>(w, a.J, r0, rk.group0, rk.n_groups, nothing_of);
}

// LONG: one GLOBAL ranking, a long list.
template <bool LC, bool VEC, bool LONG>
__global__ __launch_bounds__(kListThreads, 8) void k_begin_sample(BeginSampleArgs b, ListArgs w) {
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
    auto kept_of = [&](int j, u64 n) {                     // as the host rounds: llround of the binary64 product, clamped
        const u64 k = static_cast<u64>(llround(b.density[j] * static_cast<double>(n)));
        return k > n ? n : k;
    };
    if (blockIdx.x == 0) {
        upload_words(b.up, tid, kListThreads);
        __syncthreads();                                   // every load has returned: its value went into a store
        if (tid == 0) store_ticket(b.up.done, b.up.ticket);
        return;
    }
    const u32 block = blockIdx.x - 1;
    if (block >= b.groups + b.fillers) {                   // a population's bounds, from what the workgroups before it leave
        const u32 g = block - b.groups - b.fillers;
        const u32 group0 = b.per_tensor ? b.group0[g] : 0u, W = b.per_tensor ? b.group0[g + 1] - group0 : b.groups;
        const u64 n_pop = b.per_tensor ? b.n[g] : b.N;
        if (W != 1) list_bounds<true, LONG>(w, b.J, static_cast<u64>(g) * b.J, group0, W, [&](u32 j) { return kept_of(static_cast<int>(j), n_pop) == 0; });
        return;
    }
    if (tid <= b.n_tensors) s_start[tid] = b.chunk_start[tid];
    if (block < b.groups) {
        __shared__ const float* s_w[kBeginSampleTensors];
        __shared__ const float* s_lam[kBeginSampleTensors];
        __shared__ u32 s_n[kBeginSampleTensors];
        if (tid < b.n_tensors) {
            s_w[tid] = b.w[tid];
            s_n[tid] = b.n[tid];
            if (LC) s_lam[tid] = b.lam[tid];
        }
        __syncthreads();
        u32 g = 0, W = b.groups, me = block;
        u32 first_chunk = 0, quads = b.n_chunks * (kChunk / 4);
        u64 n_pop = b.N;
        if (b.per_tensor) {
            int lo = 0, hi = b.n_tensors - 1;              // the tensor this workgroup samples: the last with group0 <= its number
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (b.group0[mid] <= block) lo = mid; else hi = mid - 1;
            }
            g = static_cast<u32>(lo);
            W = static_cast<u32>(b.group0[g + 1]) - b.group0[g];
            me = block - b.group0[g];
            first_chunk = s_start[g];
            n_pop = s_n[g];
            quads = (s_n[g] + 3u) / 4;
        }
        list_sample<LC, VEC>(w, b.J, b.mu, W, me, block, static_cast<u64>(g) * b.J, first_chunk, quads,
                             [&](u32 c) {
                                 const int t = b.per_tensor ? static_cast<int>(g) : tensor_of_chunk_lds(c);
                                 return SampleTensor{s_w[t], LC ? s_lam[t] : nullptr, s_n[t], s_start[t]};
                             },
                             [&](int j, u64* k, u64* n) { *k = kept_of(j, n_pop); *n = n_pop; });
        return;
    }
    __syncthreads();
    const u64 stride = static_cast<u64>(b.fillers) * kListThreads;
    const u64 i0 = static_cast<u64>(block - b.groups) * kListThreads + tid;
    const uint4 z = make_uint4(0, 0, 0, 0);
    for (u64 i = i0; i < b.n_zero; i += stride) b.zero[i] = z;
    for (u64 c = i0; c < b.n_chunks; c += stride) b.chunk_map[c] = static_cast<u32>(tensor_of_chunk_lds(static_cast<u32>(c)));
}

__device__ inline u32 lanes_below(u64 m) {       // set bits of m below this lane's
    return __builtin_amdgcn_mbcnt_hi(static_cast<u32>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<u32>(m), 0));
}

// Where this workgroup counts ranking r's listed keys.  A line that many update takes some 10 ns for each of them, so there are
// up to 16 copies, taken in turn, and 64 where the keys may meet in few bins (pruning VGG-19 at a gap, some 100 thousand keys in a
// few bins: the sweep 70 us with 16 copies, 38 with 64, 32 where it does not count them; on 8-bit integers 44, 33 and 31).
__device__ inline u32 list_copies(const ListArgs& w, const ListWin& win) { return win_uneven(win) ? w.uneven_copies : w.hist_copies; }
__device__ inline u32* list_hist(const ListArgs& w, u64 r) { return w.hist + r * w.uneven_copies * kListBins; }
__device__ inline u32* list_hist_copy(const ListArgs& w, u64 r, const ListWin& win) {
    return list_hist(w, r) + (blockIdx.x & (list_copies(w, win) - 1)) * kListBins;
}

// Counts of a wavefront's listed keys.  A few go straight to the histogram.  Where they are many, those of the first two bins met are
// added up first: they may be equal (five layers of 2.4 M E4M3 values: 130 thousand updates of one counter; 595 us the call
// without, 240 with).
constexpr u32 kCountedAtOnce = 8;
struct BinCounts {
    u32 bin[2] = {0, 0}, n[2] = {0, 0};          // uniform
    __device__ inline void add(u32* hist, bool there, u32 b) {           // all lanes
        u64 rest = __ballot(there);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (rest == 0) return;               // uniform
            if (n[i] == 0) bin[i] = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(b), __ffsll(static_cast<long long>(rest)) - 1));
            const u64 same = __ballot(there && b == bin[i]) & rest;
            n[i] += static_cast<u32>(__popcll(same));
            rest &= ~same;
        }
        if ((rest >> (threadIdx.x & 63u)) & 1u) atomicAdd(hist + b, 1u);
    }
    __device__ inline void flush(u32* hist) const {
        const u32 lane = threadIdx.x & 63u, mine = lane == 0 ? n[0] : n[1];
        if (lane < 2 && mine) atomicAdd(hist + (lane == 0 ? bin[0] : bin[1]), mine);
    }
};

// ---- the one pass over the weights: one density ------------------------------------------------------------
//
// As k_window_fused, with one list per ranking and one counter update per wavefront (entries and keys above the window in
// the halves of a word; they stay right when the list is full).  One float4 per lane and array for the L-C forms, four for pruning (measured there).
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
    if (win_crowded(win)) return;                                       // uniform
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
    u32 inside = 0;                                                     // a bit for each of this lane's elements that is inside the window
    u32 above = 0, nz = 0;                                              // sums over the wavefront
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
            const bool hit = in && x - lo <= span;
            inside |= hit ? 1u << (4 * q + k) : 0u;
            above += static_cast<u32>(__popcll(__ballot(keep && in && !hit)));                  // the estimate lies in the window
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
    const u32 mine = static_cast<u32>(__popc(inside)), incl = wave_incl_scan_u32(mine);
    const u32 total = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
    if ((total | above) == 0) return;
    u64 b = 0;
    if (lane == 0)
        b = atomicAdd(reinterpret_cast<unsigned long long*>(&w.cnt[static_cast<u64>(r) * w.max_segs + seg]),
                      (static_cast<unsigned long long>(above) << 32) | total);
    if (total == 0) return;
    u32* const hist = w.count_in_sweep ? list_hist_copy(w, r, win) : nullptr;
    const u32 shift = win_shift(win);
    const bool add_up = total > kCountedAtOnce || win_uneven(win);
    BinCounts counts;
    u32 at = incl - mine;
    const u64 first = rk.base + static_cast<u64>(seg) * rk.seg_cap;
    const u32 i0 = static_cast<u32>(c) * kChunk + sub * kWaveElems + lane * 4, pos = __shfl(static_cast<u32>(b), 0, 64);
    while (__any(inside != 0)) {                                        // every lane its next element (one or two of them, as a rule)
        const bool there = inside != 0;
        const u32 i = there ? static_cast<u32>(__ffs(inside)) - 1u : 0u;
        inside &= inside - 1u;
        u32 x = key[0][0];
#pragma unroll
        for (int e = 1; e < 4 * QUADS; ++e) x = i == static_cast<u32>(e) ? key[e / 4][e % 4] : x;
        if (hist) {                                                     // uniform
            if (add_up) counts.add(hist, there, (x - lo) >> shift);
            else if (there)             atomicAdd(hist + ((x - lo) >> shift), 1u);
        }
        if (there && pos + at < rk.seg_cap) {
            w.key[first + pos + at] = x;
            w.idx[first + pos + at] = i0 + (i >> 2) * 256 + (i & 3u);
        }
        ++at;
    }
    if (hist) counts.flush(hist);
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
constexpr u32 kListMultiBuf = 256;               // buffered entries of a wavefront, of all rankings; with more, they come from the tile
struct ListMultiShared {
    u32 tile[256 * kListMultiQuads];             // the tile's keys, then its regions
    u32 key[kListMultiBuf];
    u32 what[kListMultiBuf];                     // element of the tile | ranking << 12 | place among the ranking's entries << 16
    u32 count[kMaxJ];                            // entries | those from the estimate on << 16
    u32 gap[2 * (kMaxJ + 1)];
    u32 ranking[kMaxJ];
};
static_assert(256 * kListMultiQuads <= 1 << 12 && kMaxJ <= 16, "ListMultiShared::what");

__device__ inline u32 list_reserve(const ListArgs& w, u64 r, const ListRank& rk, u32 count, u32 above) {
    return static_cast<u32>(atomicAdd(reinterpret_cast<unsigned long long*>(&w.cnt[r * w.max_segs + blockIdx.x % rk.n_segs]),
                                      (static_cast<unsigned long long>(above) << 32) | count));
}
// `mine`: in lane j, ranking j's buffered entries and (upper half) its keys above the window; `total`: the entries of all.  A lane takes an
// entry, whatever its ranking (one ranking after the other, the ten of a search cost a wavefront 250 instructions).
__device__ inline void list_multi_flush(const DataArgs& a, const ListArgs& w, const ListMultiShared& sh, u64 r0, u64 mine, u32 total, u32 i0) {
    const int lane = threadIdx.x;
    ListRank rk{};
    u32 at = 0;
    if (lane < a.J && mine) {
        rk = w.rank[r0 + lane];
        at = list_reserve(w, r0 + lane, rk, static_cast<u32>(mine), static_cast<u32>(mine >> 32));
    }
    const u64 first = rk.base + (rk.n_segs ? static_cast<u64>(blockIdx.x % rk.n_segs) * rk.seg_cap : 0) + at;
    const u32 room = at < rk.seg_cap ? rk.seg_cap - at : 0u;
    __syncthreads();                                                    // one wavefront: orders the LDS buffer
    for (u32 e0 = 0; e0 < total; e0 += 64) {                            // uniform
        const u32 e = e0 + lane, what = e < total ? sh.what[e] : 0u, i = what >> 16;
        const int j = static_cast<int>((what >> 12) & 15u);
        const u64 to = ((static_cast<u64>(__shfl(static_cast<u32>(first >> 32), j, 64)) << 32) | __shfl(static_cast<u32>(first), j, 64)) + i;
        const bool fits = i < __shfl(room, j, 64);
        if (e < total && fits) {
            w.key[to] = sh.key[e];
            w.idx[to] = i0 + (what & 0xFFFu);
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
    u64 mine = 0;                                                       // lane j: ranking j's buffered entries and keys above
    u32 total = 0;
    for (int j = 0; j < a.J; ++j) {
        const ListWin win = w.win[r0 + j];
        if (win_crowded(win)) continue;                                 // uniform
        const u32 lo = win.lo, span = win.hi - win.lo, mid = win.mid;
        OutDesc o{};
        if (w.write) o = w.out[static_cast<u64>(j) * a.n_tensors + t];
        u32 count = 0, above = 0;
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
                m[k] = keep ? 1 : 0;
                th[k] = keep ? v[q][k] : 0.0f;
                const u64 hit = __ballot(there && x - lo <= span);
                above += static_cast<u32>(__popcll(__ballot(keep && there) & ~hit));
                if (hit != 0) {                                         // uniform
                    const u32 n_hit = static_cast<u32>(__popcll(hit));
                    const bool me = (hit >> lane) & 1u;
                    if (total + n_hit <= kListMultiBuf) {
                        if (me) {
                            sh.key[total + lanes_below(hit)] = x;
                            sh.what[total + lanes_below(hit)] = static_cast<u32>(q * 256 + lane * 4 + k) | static_cast<u32>(j) << 12 | (count + lanes_below(hit)) << 16;
                        }
                        count += n_hit;
                        total += n_hit;
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
        if (lane == j) mine = (static_cast<u64>(above) << 32) | count;
    }
    list_multi_flush(a, w, sh, r0, mine, total, i0);
}

// WIDE: masks only, each 16-byte aligned.
// Bound by instructions (ten densities: 980 for a wavefront's 1024 elements, 1214 before) and the latency of what a wavefront waits for, with six of them
// on a SIMD: outputs, estimates and biases of all rankings are loaded at once, a lane each, and counts cross the lanes two to a sum in registers.
// Ten masks of 20 M weights 76 -> 53 us, the call 123 -> 104; of 113 M weights, the call 501 -> 354, two densities of them 235 -> 193.
template <bool VEC, bool WIDE, int Q>
__global__ __launch_bounds__(64, WIDE || Q == 1 ? 6 : 5) void k_list_sweep_multi(DataArgs a, ListArgs w) {
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
    if (srt.idle) return;                                               // uniform
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
    // What the loops over rankings need is loaded by a lane each, now, and read across lanes there.
    const u32 mid_of = lane < kMaxJ ? srt.mid[lane < kMaxJ ? lane : 0] : 0u, bias_of = lane < kMaxJ ? srt.bias[lane < kMaxJ ? lane : 0] : 0u;
    OutDesc out_of{};
    if (w.write && lane < a.J) out_of = w.out[static_cast<u64>(lane) * a.n_tensors + t];
    if (lane < kMaxJ) { sh.count[lane] = 0; sh.ranking[lane] = srt.ranking[lane]; }
    if (lane <= kMaxJ) { sh.gap[2 * lane] = srt.gap_lo[lane]; sh.gap[2 * lane + 1] = srt.gap_len[lane]; }
    u32 region[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) region[q][k] = 0;
    for (u32 p = 0; p < n; ++p) {
        const u32 mid = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(mid_of), static_cast<int>(p)));       // uniform
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
    const u32 i0 = static_cast<u32>(c) * kChunk + sub * kWaveElems;
    u32 total = 0;                                                      // uniform
    for (u64 left; (left = __ballot(inside != 0)) != 0;) {              // uniform
        if (inside) {
            const u32 i = static_cast<u32>(__ffs(inside)) - 1u, off = (i >> 2) * 256 + lane * 4 + (i & 3u);
            inside &= inside - 1u;
            u32 word = packed[0];
#pragma unroll
            for (int q = 1; q < Q; ++q) word = (i >> 2) == static_cast<u32>(q) ? packed[q] : word;
            const u32 r = (word >> (8 * (i & 3u))) & 0xFFu, x = sh.tile[off];
            // below the gap of its region: the window of the highest estimate it reaches; else the next one up
            const bool reaches = x < sh.gap[2 * r];
            const u32 j = sh.ranking[reaches ? n - r : n - r - 1u];
            const u32 at = atomicAdd(&sh.count[j], reaches ? 0x10001u : 1u) & 0xFFFFu, e = total + lanes_below(left);
            if (e < kListMultiBuf) {
                sh.key[e] = x;
                sh.what[e] = off | j << 12 | at << 16;
            }
        }
        total += static_cast<u32>(__popcll(left));
    }
    const bool buffered = total <= kListMultiBuf;                       // uniform
    u64 from_tile = buffered ? 0 : __ballot(lane < a.J && (sh.count[lane < a.J ? lane : 0] & 0xFFFFu) != 0);
    while (from_tile != 0) {                                            // uniform.  All of that ranking's entries from the tile
        const u32 j = static_cast<u32>(__ffsll(static_cast<long long>(from_tile))) - 1u;
        from_tile &= from_tile - 1u;
        const ListWin win = w.win[r0 + j];
        const ListRank rk = w.rank[r0 + j];
        u32 pos = 0;
        if (lane == 0) pos = list_reserve(w, r0 + j, rk, sh.count[j] & 0xFFFFu, 0);
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
    auto pointer_of = [](const void* p, int j) {                        // lane j's, in all lanes
        const u64 x = reinterpret_cast<u64>(p);
        return reinterpret_cast<void*>((static_cast<u64>(static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(x >> 32), j))) << 32) |
                                       static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(x), j)));
    };
    u32 kept_of_lane = 0, kept_pair = 0;                                // lane j: ranking j's keys from its estimate on
    for (int j = 0; j < a.J; ++j) {
        const u32 bias = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(bias_of), j)) * 0x01010101u;
        u8* const mask = static_cast<u8*>(pointer_of(out_of.mask, j));
        u32 m[Q], kept = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            m[q] = ((packed[q] + bias) >> 7) & 0x01010101u;
            kept = __builtin_amdgcn_udot4(m[q], 0x01010101u, kept, false);
        }
        if constexpr (WIDE) {
            if (mask) {
                u32x4 t4;
                t4.x = m[0]; t4.y = m[1]; t4.z = m[2]; t4.w = m[3];
                st_words4_stream(mask + base, static_cast<u32>(lane) * 16u, t4);
            }
        } else {
            float* const theta = static_cast<float*>(pointer_of(out_of.theta, j));
            u16* const theta16 = static_cast<u16*>(pointer_of(out_of.theta16, j));
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const u64 e0 = base + q * 256 + lane * 4;
                if (mask) st_mask4_stream(mask + e0, static_cast<u8>(m[q] & 1u), static_cast<u8>((m[q] >> 8) & 1u),
                                          static_cast<u8>((m[q] >> 16) & 1u), static_cast<u8>(m[q] >> 24));
                if (!theta && !theta16) continue;
                float th[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) th[k] = ((m[q] >> (8 * k)) & 1u) ? v[q][k] : 0.0f;
                if (theta) st4_stream(theta + e0, th[0], th[1], th[2], th[3]);
                if (theta16)
                    st_code4_stream(theta16 + e0, f32_to_f16_rne(th[0]), f32_to_f16_rne(th[1]), f32_to_f16_rne(th[2]), f32_to_f16_rne(th[3]));
            }
        }
        // two rankings' counts are added up over the wavefront together (at most 1024 each)
        kept_pair |= kept << (16 * (j & 1));
        if ((j & 1) == 0 && j + 1 < a.J) continue;
        const u32 sums = wave_sum_u32(kept_pair);
        kept_pair = 0;
        if (lane == (j & ~1)) kept_of_lane = sums & 0xFFFFu;
        if (lane == (j | 1)) kept_of_lane = sums >> 16;
    }
    __syncthreads();
    const u32 offered = lane < a.J ? sh.count[lane] & 0xFFFFu : 0u, reached = lane < a.J ? sh.count[lane] >> 16 : 0u;
    list_multi_flush(a, w, sh, r0, (static_cast<u64>(kept_of_lane - reached) << 32) | (buffered ? offered : 0u), buffered ? total : 0u, i0);
}

// ---- the threshold among the listed keys ---------------------------------------------------------------

// f(there, key, entry) for the entries of ranking s that this wavefront takes: every `stride`-th segment, kListDeep rows
// of four segments at a time (their loads in flight together); called by all lanes, `there` says which hold an entry.  The
// segments' counts come from LDS (cnt_of) where the workgroup has them.
constexpr u32 kListDeep = 4;
template <typename F>
__device__ inline void list_walk(const ListArgs& w, u32 s, const ListRank& rk, u32 first_seg, u32 stride, const u32* cnt_of, F&& f) {
    const u32 lane = threadIdx.x & 63u;
    for (u32 seg0 = first_seg; seg0 < rk.n_segs; seg0 += 64 * stride) {
        const u32 my_seg = seg0 + lane * stride;
        u32 my_cnt = 0;
        if (my_seg < rk.n_segs) my_cnt = cnt_of ? cnt_of[my_seg] : static_cast<u32>(w.cnt[static_cast<u64>(s) * w.max_segs + my_seg]);
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

// f(there, key, index) for the entries of the ranking that this wavefront takes: every `stride`-th segment, `cnt` entries each (in
// LDS), kListDeep rows of two segments at a time with their loads in flight together; called by all lanes, `there` says which hold
// an entry.
template <typename F>
__device__ inline void list_walk_own(const ListArgs& w, const ListRank& rk, const u32* cnt_of, u32 first_seg, u32 stride, F&& f, u32 part = 0, u32 parts = 1) {
    const u32 lane = threadIdx.x & 63u;
    for (u32 seg0 = first_seg; seg0 < rk.n_segs; seg0 += 2 * stride) {
        u32 cnt[2], most = 0;
        u64 first[2];
#pragma unroll
        for (u32 b = 0; b < 2; ++b) {
            const u32 seg = seg0 + b * stride;
            cnt[b] = seg < rk.n_segs ? cnt_of[seg] : 0u;
            first[b] = rk.base + static_cast<u64>(seg) * rk.seg_cap;
            most = cnt[b] > most ? cnt[b] : most;
        }
        for (u32 i0 = 64 * kListDeep * part; i0 < most; i0 += 64 * kListDeep * parts) {              // uniform
            u32 x[kListDeep][2], e[kListDeep][2];
#pragma unroll
            for (u32 d = 0; d < kListDeep; ++d)
#pragma unroll
                for (u32 b = 0; b < 2; ++b) {
                    const u32 i = i0 + 64 * d + lane, last = cnt[b] ? cnt[b] - 1u : 0u;
                    const u64 at = first[b] + (i < cnt[b] ? i : last);
                    if (i0 + 64 * d < cnt[b]) { x[d][b] = w.key[at]; e[d][b] = w.idx[at]; }        // uniform
                }
#pragma unroll
            for (u32 d = 0; d < kListDeep; ++d)
#pragma unroll
                for (u32 b = 0; b < 2; ++b)
                    if (i0 + 64 * d < cnt[b]) f(i0 + 64 * d + lane < cnt[b], x[d][b], e[d][b]);    // uniform
        }
    }
}

// hist[bin] += 1 for the lanes that are `there`; all lanes call it.  Lanes that meet on a counter take turns, and listed keys
// often are equal (weights on a grid), so the two commonest-looking bins are added up across the wavefront first.
__device__ inline void wave_count(u32* hist, bool there, u32 bin) {
    u64 rest = __ballot(there);
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        if (rest == 0) return;                             // uniform
        const int leader = __ffsll(static_cast<long long>(rest)) - 1;
        const u32 b = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(bin), leader));
        const u64 same = __ballot(there && bin == b);
        if (static_cast<int>(threadIdx.x & 63u) == leader) atomicAdd(&hist[b], static_cast<u32>(__popcll(same)));
        there = there && bin != b;
        rest &= ~same;
    }
    if (there) atomicAdd(&hist[bin], 1u);
}

// Counts of a ranking's listed keys per bin of its window, where the sweep did not take them; `parts` workgroups per ranking.
__global__ __launch_bounds__(kBlock) void k_list_hist(ListArgs w) {
    constexpr int kCopies = 8;                             // by lane: listed keys often are equal (weights on a grid), and lanes
    __shared__ __align__(16) u32 s_hist[kListBins * kCopies];            // that meet on a counter take turns
    const u32 s = blockIdx.x / w.parts, part = blockIdx.x % w.parts;
    const ListRank rk = w.rank[s];
    const ListWin win = w.win[s];
    const u32 wave = threadIdx.x >> 6, first = part * (kBlock / 64) + wave, stride = w.parts * (kBlock / 64);
    if (part * (kBlock / 64) >= rk.n_segs || win_crowded(win)) return;   // uniform: nothing for this workgroup
    for (u32 i = threadIdx.x; i < static_cast<u32>(kListBins * kCopies) / 4; i += kBlock) reinterpret_cast<uint4*>(s_hist)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    const u32 lo = win.lo, shift = win_shift(win), copy = threadIdx.x & (kCopies - 1);
    list_walk(w, s, rk, first, stride, nullptr, [&](bool there, u32 key, u64) {
        if (there) atomicAdd(&s_hist[((key - lo) >> shift) * kCopies + copy], 1u);
    });
    __syncthreads();
    const uint4 v0 = reinterpret_cast<const uint4*>(s_hist)[2 * threadIdx.x], v1 = reinterpret_cast<const uint4*>(s_hist)[2 * threadIdx.x + 1];
    const u32 v = v0.x + v0.y + v0.z + v0.w + v1.x + v1.y + v1.z + v1.w;          // kListBins == kBlock
    if (v) atomicAdd(list_hist_copy(w, s, win) + threadIdx.x, v);
}

// The outputs of up to B listed elements, with the decision each should have had: what has to be read (list_fix_load), which need
// not wait for the decision, and the stores.  The dependent loads of the elements (tensor, its pointers, the inputs) are issued
// side by side: one after the other they take some 3 us an element.
template <bool LC, int B>
struct FixLoads {
    float wv[B], lv[B];
    float* lo[B];
    float* gr[B];
    u64 e[B];
    OutDesc o[B];
};
template <bool LC, int B>
__device__ inline void list_fix_load(const DataArgs& a, const ListArgs& w, u32 j, const u32 (&idx)[B], const bool (&on)[B], FixLoads<LC, B>& x) {
    u32 t[B];
#pragma unroll
    for (int b = 0; b < B; ++b) t[b] = on[b] ? a.chunk_map[idx[b] / kChunk] : 0u;
    const float* wp[B];
    const float* lp[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const TensorDesc& td = a.td[t[b]];
        wp[b] = td.w;
        if (LC) { lp[b] = td.lam; x.lo[b] = td.lam_out; x.gr[b] = td.grad; }
        x.e[b] = static_cast<u64>(idx[b]) - td.chunk_start * kChunk;
        x.o[b] = w.out[static_cast<u64>(j) * a.n_tensors + t[b]];
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        x.wv[b] = on[b] ? wp[b][x.e[b]] : 0.0f;
        x.lv[b] = LC && on[b] ? lp[b][x.e[b]] : 0.0f;
    }
}
template <bool LC, bool PQ, int B>
__device__ inline void list_fix_store(const DataArgs& a, const FixLoads<LC, B>& x, const bool (&keep)[B], const bool (&on)[B], int* nz) {
#pragma unroll
    for (int b = 0; b < B; ++b) {
        if (!on[b]) continue;
        const OutDesc& o = x.o[b];
        const u64 e = x.e[b];
        if (LC) {
            const float v = lc_shift(x.wv[b], x.lv[b], a.mu);
            float th = keep[b] ? v : 0.0f;
            if (PQ) {
                const u16 hv = f32_to_f16_rne(v), h = keep[b] ? hv : static_cast<u16>(0);
                th = f16_bits_to_f32(h);
                if (o.theta16) o.theta16[e] = h;
                if ((hv & 0x7FFFu) != 0) *nz += keep[b] ? 1 : -1;
            }
            const float p = __fmul_rn(a.mu, __fsub_rn(x.wv[b], th));
            const float ln = __fsub_rn(x.lv[b], p);
            if (o.theta) o.theta[e] = th;
            x.lo[b][e] = ln;
            if (x.gr[b]) x.gr[b][e] = __fsub_rn(p, ln);
        } else {
            const float th = keep[b] ? x.wv[b] : 0.0f;
            if (o.theta) o.theta[e] = th;
            if (o.theta16) o.theta16[e] = f32_to_f16_rne(th);
        }
        if (o.mask) o.mask[e] = keep[b] ? 1 : 0;
    }
}
template <bool LC, bool PQ, int B>
__device__ inline void list_fix(const DataArgs& a, const ListArgs& w, u32 j, const u32 (&idx)[B], const bool (&keep)[B], const bool (&on)[B], int* nz) {
    FixLoads<LC, B> x;
    list_fix_load<LC, B>(a, w, j, idx, on, x);
    list_fix_store<LC, PQ, B>(a, x, keep, on, nz);
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

__device__ inline void st_state(ListState* to, u32 a, u32 b, u32 rank, u32 n, u32 flags) {
    st_dev(&to->a, a); st_dev(&to->b, b); st_dev(&to->rank, rank); st_dev(&to->n, n); st_dev(&to->flags, flags);
}
__device__ inline ListState ld_state(const ListState* from) {
    ListState x{};
    x.a = ld_dev(&from->a); x.b = ld_dev(&from->b); x.rank = ld_dev(&from->rank); x.n = ld_dev(&from->n); x.flags = ld_dev(&from->flags);
    return x;
}

// Where a threshold is that is not in its list, or whose list is incomplete: `inside` keys in the window, `above` above it, all
// counted by the sweep.
__device__ inline ListState list_window_state(const ListWin& win, u32 n, u32 k, u32 above, u32 inside) {
    ListState x{};
    if (above >= k)               { x.a = win.hi + 1u; x.b = 0x7FFFFFFFu; x.rank = k; x.n = above; }
    else if (k - above <= inside) { x.a = win.lo; x.b = win.hi; x.rank = k - above; x.n = inside; }
    else                          { x.a = 0; x.b = win.lo - 1u; x.rank = k - above - inside; x.n = n - above - inside; }
    return x;
}
// Ranking s goes to list_fallback: `rank` from the top between a and b, where there are n keys.  All threads of one
// workgroup; its histogram is cleared here.
template <int THREADS>
__device__ inline void list_leave(const DataArgs& a, const ListArgs& w, u32 s, u32 lo, u32 hi, u32 rank, u32 n, u32 flags) {
    for (u32 i = threadIdx.x; i < 3 * w.fb_bins; i += THREADS) st_dev(w.fb_hist + static_cast<u64>(s) * 3 * w.fb_bins + i, 0u);
    if (threadIdx.x != 0) return;
    const u32 g = s / a.J, j = s - g * a.J;
    st_dev(w.fb_above + s, 0u);
    st_state(w.state + s, lo, hi, rank, n, flags);
    st_dev(w.special + add_dev(&w.fb->special, 1u), s);
    if (flags & kStateMaybe) {
        if (rank < n) or_dev(w.tie_of + g, 1u << j);
        return;
    }
    add_dev(&w.fb->apply, 1u);
    or_dev(w.apply_of + g, 1u << j);
    if (lo < hi || (flags & kStateUnsure)) {
        or_dev(w.open_of + g, 1u << j);
        add_dev(&w.fb->open[0], 1u);
    } else if (rank < n) {
        or_dev(w.tie_of + g, 1u << j);
        add_dev(&w.fb->ties, 1u);
    }
}
// Where the threshold of ranking s is in its list, from the counters and the histogram that the sweep left.  All threads; every
// workgroup of the ranking finds the same, and every wavefront of it once the copies of the histogram are added up.  The loads depend
// on nothing but the launch's arguments and are all in flight at once.
template <int THREADS>
struct ListFindShared {
    u32 cnt[kListSegs];    // entries of each segment
    uint4 hist[THREADS / 64][64];                // sums over a wavefront's copies, four bins a lane, from the top
    u32 above[THREADS / 64], listed[THREADS / 64], over[THREADS / 64], scratch[THREADS / 64];
};
struct ListFound {
    u32 above, listed;     // keys above the window and in it
    u32 bin, want, n_in;   // the threshold's bin, its rank among the keys there, their number.  want 0: it is not in the list, or
                           // the list is not complete
};
template <int THREADS>
__device__ inline ListFound list_find(const ListArgs& w, ListFindShared<THREADS>& sh, u32 s, const ListRank& rk, const ListWin& win, u32 k) {
    static_assert(kListSegs % THREADS == 0 && kListBins == 4 * 64, "segments by thread, bins by lane");
    constexpr int kPer = kListSegs / THREADS;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    u64 v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const u32 seg = tid + i * THREADS;
        v[i] = seg < w.max_segs ? w.cnt[static_cast<u64>(s) * w.max_segs + seg] : 0;           // none past n_segs
    }
    uint4 h = make_uint4(0, 0, 0, 0);
    const u32* from = list_hist(w, s) + (kListBins - 4 - 4 * lane);
    auto add_copy = [&](u32 c) {
        const uint4 x = *reinterpret_cast<const uint4*>(from + c * kListBins);
        h.x += x.x; h.y += x.y; h.z += x.z; h.w += x.w;
    };
#pragma unroll 2
    for (u32 c = wave; c < w.hist_copies; c += THREADS / 64) add_copy(c);
    if (win_uneven(win))                                   // uniform; the others do not wait for the window
#pragma unroll 6
        for (u32 c = w.hist_copies + wave; c < w.uneven_copies; c += THREADS / 64) add_copy(c);
    sh.hist[wave][lane] = h;
    u32 above = 0, listed = 0;
    bool over = false;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const u32 n = static_cast<u32>(v[i]);
        above += static_cast<u32>(v[i] >> 32);             // neither sum reaches 2^32
        listed += n;
        over = over || n > rk.seg_cap;
        sh.cnt[tid + i * THREADS] = n < rk.seg_cap ? n : rk.seg_cap;
    }
    above = wave_sum_u32(above);
    listed = wave_sum_u32(listed);
    const bool any_over = __any(over);
    if (lane == 63) { sh.above[wave] = above; sh.listed[wave] = listed; sh.over[wave] = any_over ? 1u : 0u; }
    __syncthreads();
    ListFound f{};
    u32 any = 0;
    h = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (u32 i = 0; i < THREADS / 64; ++i) {
        f.above += sh.above[i];
        f.listed += sh.listed[i];
        any |= sh.over[i];
        const uint4 x = sh.hist[i][lane];
        h.x += x.x; h.y += x.y; h.z += x.z; h.w += x.w;
    }
    const u32 c[4] = {h.w, h.z, h.y, h.x}, sum = h.x + h.y + h.z + h.w, incl = wave_incl_scan_u32(sum);
    const u32 want = k - f.above;                          // (when that many are above, nothing below holds)
    u32 before = incl - sum, bin = 0, rem = 0, in = 0;
    const u64 here = __ballot(any == 0 && f.above < k && before < want && want <= incl);
    if (here == 0) return f;                               // uniform
#pragma unroll
    for (u32 i = 0; i < 4; ++i) {
        if (before < want && want <= before + c[i]) { bin = kListBins - 1 - 4 * lane - i; rem = want - before; in = c[i]; }
        before += c[i];
    }
    const int at = __ffsll(static_cast<long long>(here)) - 1;
    f.bin = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(bin), at));
    f.want = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(rem), at));
    f.n_in = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(in), at));
    return f;
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
        const u32 sum = c[0] + c[1] + c[2] + c[3], incl = wave_incl_scan_u32(sum);
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
// number 0 writes state and record.  What they read of the ranking's state is never written here.  SAME: other workgroups of
// this launch gathered the entries; their loads pass the caches, so several are in flight at a time.
template <bool LC, bool PQ, int THREADS, bool SAME>
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
        const u32* gkey = w.gkey + static_cast<u64>(s) * w.gather_cap;
        const u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
        auto ld_gathered = [](const u32* p) { if constexpr (SAME) return ld_dev(p); else return *p; };
        if (!in_lds && n <= kListRanked) {
            for (u32 i = tid; i < n; i += THREADS) { sh.key[i] = ld_gathered(gkey + i); sh.idx[i] = ld_gathered(gidx + i); }
            in_lds = true;
        }
        auto key_of = [&](u32 i) { return in_lds ? sh.key[i] : ld_gathered(gkey + i); };
        auto idx_of = [&](u32 i) { return in_lds ? sh.idx[i] : ld_gathered(gidx + i); };
        auto for_keys = [&](auto&& f) {                    // f(there, i, key) for this thread's entries; called by all lanes
            constexpr u32 kAhead = SAME ? 8 : 1;
            for (u32 i0 = 0; i0 < n; i0 += kAhead * THREADS) {           // uniform
                u32 key[kAhead];
#pragma unroll
                for (u32 b = 0; b < kAhead; ++b) { const u32 i = i0 + b * THREADS + tid; key[b] = i < n ? key_of(i) : 0u; }
#pragma unroll
                for (u32 b = 0; b < kAhead; ++b) { const u32 i = i0 + b * THREADS + tid; f(i < n, i, key[b]); }
            }
        };
        if (tid == 0) sh.r = 0;
        __syncthreads();
        // The threshold is one of the keys from .. from + 2^bits - 1: of the window's bin, or of the gathered keys' range where that
        // was kept (many may lie in a small part of the bin).  Levels of 256 bins until all pairs of the rest can be compared or
        // they are equal.  (17 rankings of VGG-19 at a gap, some 20 thousand entries each: 136 us with eight bits of the bin, then radix
        // levels on the whole key and the index; 57 so.)
        const ListWin win = w.win[s];
        u32 bits = win_shift(win), from = 0;
        if (THREADS != kListThreads && n > kListRanked) {
            from = ~ld_dev(w.gmaxc + s);
            bits = 32u - static_cast<u32>(__builtin_clz((ld_dev(w.gmax + s) - from) | 1u));
        } else {
            from = win.lo + (((key_of(0) - win.lo) >> bits) << bits);
        }
        u32 in_bin = n, bin;
        do {
            const u32 sub = bits > 8 ? bits - 8 : 0;
            if (tid < static_cast<u32>(kListBins)) sh.hist[tid] = 0;
            __syncthreads();
            for_keys([&](bool there, u32, u32 key) {
                const u32 b = (key - from) >> sub;
                if (in_bin != n)                                  wave_count(sh.hist, there && ((key - from) >> bits) == 0, b);
                else if (there && ((key - from) >> bits) == 0)    atomicAdd(&sh.hist[b], 1u);
            });
            __syncthreads();
            list_pick(sh, true, want, &bin, &want, &in_bin);
            from += bin << sub;
            bits = sub;
        } while (in_bin > kListPairs && bits > 0);         // uniform
        if (in_bin <= kListPairs) {                        // uniform
            for_keys([&](bool there, u32 i, u32 key) {
                if (there && ((key - from) >> bits) == 0) {
                    const u32 p = atomicAdd(&sh.r, 1u);
                    sh.pkey[p] = key;
                    sh.pidx[p] = idx_of(i);
                }
            });
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
        } else {                                           // ties: radix levels on the index, lowest first
            u32 prefix = 0, rem = want, n_eq, b;
            for (int shift = 24; shift >= 0; shift -= 8) {
                if (tid < static_cast<u32>(kListBins)) sh.hist[tid] = 0;
                __syncthreads();
                for_keys([&](bool there, u32 i, u32 key) {
                    const bool tie = there && key == from;
                    const u32 idx = tie ? idx_of(i) : 0u;
                    wave_count(sh.hist, tie && (shift == 24 || (idx >> (shift + 8)) == (prefix >> (shift + 8))), (idx >> shift) & 255u);
                });
                __syncthreads();
                list_pick(sh, false, rem, &b, &rem, &n_eq);
                prefix |= b << shift;
            }
            if (tid == 0) { sh.T = from; sh.rem = want; sh.n_tie = in_bin; sh.last = prefix; }
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
        } else if (tid == 0) {                             // one of several: corrections of what is stored
            const long long d = static_cast<int>(total) + (share == 0 ? static_cast<long long>(ld_dev64(&a.ctl->nnz_delta)) : 0ll);
            if (d != 0) __hip_atomic_fetch_add(w.nnz_out, static_cast<u64>(d), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();                                       // the shared words are free for the next ranking
}

// The same for the posted entries of k_list_resolve by the workgroup that posts last: at most kListFound, a few hundred as a rule.
// Radix levels of eight bits on the key (from the top of its bin), then on the index, until all pairs of the rest can be compared.
// The verdict goes to the workgroups that posted (one of them settling 800 entries of 44 M weights took 15 us: each touches a page
// of its own in every array); only what belongs to none, or to one that has left, is settled here.
constexpr u32 kShortPairs = 64;
struct RankShort {
    u64 entry[kListFound];                       // distance of the key from the top of its bin << 32 | index
    u64 pair[kShortPairs];
    u64 found;
    __align__(16) u32 hist[256];
    u32 bin, rem, in, n, n_tie, kept, missing[kMaxWalkers / 8];
    u8 owned[kListFound];                        // its workgroup settles it
};
// Posts are on their way when they are waited for (their workgroups are running), so this bound, some 0.1 s, is not met.  If it were, the
// workgroup would fetch the entries itself from the lists, which are whole, and settle them all: it tells nobody, so the others leave.  (1.2 G weights
// have some 2.7 M listed: a few ms.)
constexpr u32 kPostPolls = 1u << 16;
// `cnt`: entries of the list's segments, in LDS.
template <bool LC, bool PQ, int THREADS>
__device__ inline void list_rank_short(const DataArgs& a, const ListArgs& w, const ListRank& rk, const u32* cnt, RankShort& sh, u32 want, u32 n, u32 bin,
                                       const ListWin& win, u32 walkers, condensa_select* results, int* nz) {
    static_assert(THREADS >= 256 && THREADS >= static_cast<int>(kMaxWalkers), "a thread a bin, a thread a workgroup");
    const u32 tid = threadIdx.x, shift = win_shift(win), top_key = win.lo + (bin << shift) + ((1u << shift) - 1u);
    static_assert(THREADS / 64 <= static_cast<int>(kMaxWalkers / 8), "a word a wavefront");
    bool missing = (w.force & kForceNoPosts) != 0;
    u32 polls = 0;
    for (u32 i = tid; i < n && !missing; i += THREADS) {   // (one round, as a rule)
        u64 x;
        while (((x = ld_dev64(w.picked + i)) & kPicked) == 0 && !missing) { __builtin_amdgcn_s_sleep(1); missing = ++polls > kPostPolls; }
        sh.entry[i] = (static_cast<u64>(top_key - (static_cast<u32>(x >> 32) & 0x7FFFFFFFu)) << 32) | static_cast<u32>(x);
        sh.owned[i] = 0;
    }
    u32 range = 0;                               // of workgroup tid
    if (tid < walkers)
        while (((range = ld_dev(w.range + tid)) & kRangeKnown) == 0 && !missing) { __builtin_amdgcn_s_sleep(1); missing = ++polls > kPostPolls; }
    const bool any_missing = __any(missing);
    if ((tid & 63u) == 0) sh.missing[tid >> 6] = any_missing ? 1u : 0u;
    if (tid < 256) sh.hist[tid] = 0;
    if (tid == 0) { sh.n = 0; sh.n_tie = 0; sh.kept = 0; }
    __syncthreads();
    u32 is_missing = 0;
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) is_missing |= sh.missing[i];
    if (is_missing != 0) {                       // uniform
        for (u32 i = tid; i < n; i += THREADS) sh.owned[i] = 0;
        list_walk_own(w, rk, cnt, tid >> 6, THREADS / 64, [&](bool there, u32 key, u32 idx) {
            const u32 at = there && (key - win.lo) >> shift == bin ? atomicAdd(&sh.n, 1u) : n;             // n of them
            if (at < n) sh.entry[at] = (static_cast<u64>(top_key - key) << 32) | idx;
        });
        __syncthreads();
        if (tid == 0) sh.n = 0;
        __syncthreads();
    }
    u64 prefix = 0;
    u32 top = 32 + shift, in = n, r = want;      // the r-th from the bottom among the `in` entries whose bits from `top` on are the prefix
    while (in > kShortPairs && top > 0) {        // uniform
        const u32 width = top < 8 ? top : 8, low = top - width;
        for (u32 i = tid; i < n; i += THREADS)
            if ((sh.entry[i] >> top) == prefix) atomicAdd(&sh.hist[static_cast<u32>(sh.entry[i] >> low) & ((1u << width) - 1u)], 1u);
        __syncthreads();
        if (tid < 64) {                          // four bins a lane, from the bottom
            const uint4 c4 = *reinterpret_cast<const uint4*>(sh.hist + 4 * tid);
            const u32 c[4] = {c4.x, c4.y, c4.z, c4.w}, sum = c[0] + c[1] + c[2] + c[3];
            u32 before = wave_incl_scan_u32(sum) - sum;
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
                if (before < r && r <= before + c[i]) { sh.bin = 4 * tid + i; sh.rem = r - before; sh.in = c[i]; }
                before += c[i];
            }
        }
        __syncthreads();
        prefix = (prefix << width) | sh.bin;
        r = sh.rem;
        in = sh.in;
        top = low;
        if (tid < 256) sh.hist[tid] = 0;
        __syncthreads();
    }
    for (u32 i = tid; i < n; i += THREADS)
        if ((sh.entry[i] >> top) == prefix) sh.pair[atomicAdd(&sh.n, 1u)] = sh.entry[i];       // `in` of them
    __syncthreads();
    if (tid < in) {
        const u64 mine = sh.pair[tid];
        u32 less = 0;
#pragma unroll 4
        for (u32 e = 0; e < in; ++e) less += sh.pair[e] < mine ? 1u : 0u;
        if (less + 1 == r) sh.found = mine;      // entries differ: one thread
    }
    __syncthreads();
    const u64 found = sh.found;
    const u32 T = top_key - static_cast<u32>(found >> 32), last = static_cast<u32>(found);
    if (tid < walkers && is_missing == 0) {
        const u64 was = __hip_atomic_exchange(w.verdict + tid, kPicked | (static_cast<u64>(T) << 32) | last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const u32 first = range & ((1u << kRangeBits) - 1u), count = (range & ~kRangeKnown) >> kRangeBits;
        if (was != kWalkerLeft)
            for (u32 i = 0; i < count && first + i < kListFound; ++i) sh.owned[first + i] = 1;
    }
    for (u32 i = tid; i < n; i += THREADS)
        if ((sh.entry[i] >> 32) == (found >> 32)) {
            atomicAdd(&sh.n_tie, 1u);
            if (sh.entry[i] <= found) atomicAdd(&sh.kept, 1u);
        }
    __syncthreads();
    if (w.write)
        for (u32 i = tid; i < n; i += THREADS) {
            const bool kept = sh.entry[i] <= found;
            if (!sh.owned[i] && kept != (top_key - static_cast<u32>(sh.entry[i] >> 32) >= win.mid))
                list_fix_one<LC, PQ>(a, w, 0, static_cast<u32>(sh.entry[i]), kept, nz);
        }
    if (tid == 0) {
        Slot& slot = a.slots[0];
        u64 tie_end = slot.n;
        if (sh.kept < sh.n_tie) {
            const TensorDesc& td = a.td[a.chunk_map[last / kChunk]];
            tie_end = static_cast<u64>(last) - td.chunk_start * kChunk + (a.per_tensor ? 0 : td.flat_start) + 1;
        }
        slot.prefix = T; slot.remaining = sh.kept; slot.n_tie = sh.n_tie; slot.need_tie = 0; slot.tie_end = tie_end; slot.state = kDone;
        *results = select_record(slot, true, T, sh.kept, sh.n_tie, tie_end, is_missing == 0 ? slot.path : 3);
    }
}

// The same for long lists (k_list_resolve<..., LONG>), whose bins hold thousands of entries: up to kListPosted of them, of which LDS holds those that share
// the threshold's first digits.  1.2 G weights pruned, 12 thousand in the bin: the launch 57 us, 130 where such bins were left to the whole grid, 155
// where every digit was a pass over the posted entries.  Up to 65 536 and not 16 384: the same call with 20 thousand 1834 -> 1770 us; 604 M weights in rows of
// very different sizes, L-C step 2145 -> 2033.  A kernel of its own: with this in the one for short lists the L-C step of 20 M weights took 3.6 us more.
struct RankLong {
    u64 entry[kListFound];                       // as in RankShort
    u64 pair[kShortPairs];
    u64 found;
    __align__(16) u32 hist[256];
    u32 bin, rem, in, n, n_tie, kept, n_owned, missing[16];
    u32 owned[kListPosted / 32];                 // a bit each: its workgroup settles it
};
template <bool LC, bool PQ, int THREADS>
__device__ inline void list_rank_long(const DataArgs& a, const ListArgs& w, const ListRank& rk, const u32* cnt, RankLong& sh, u32 want, u32 n, u32 bin,
                                      const ListWin& win, u32 walkers, condensa_select* results, int* nz) {
    static_assert(THREADS >= 256 && THREADS >= static_cast<int>(kMaxWalkers * kListParts), "a thread a bin, a thread a workgroup");
    const u32 tid = threadIdx.x, shift = win_shift(win), top_key = win.lo + (bin << shift) + ((1u << shift) - 1u);
    static_assert(THREADS / 64 <= 16, "a word a wavefront");
    const bool in_lds = n <= kListFound;         // uniform
    auto entry = [&](u64 x) { return (static_cast<u64>(top_key - (static_cast<u32>(x >> 32) & 0x7FFFFFFFu)) << 32) | static_cast<u32>(x); };
    const u64* from = w.picked;
    // f(place, entry) for all that were posted, eight loads at a time (they pass the caches)
    auto posted = [&](auto&& f) {
        for (u32 i0 = tid; i0 < n; i0 += 8 * THREADS) {
            u64 x[8];
#pragma unroll
            for (u32 j = 0; j < 8; ++j) x[j] = ld_dev64(from + (i0 + j * THREADS < n ? i0 + j * THREADS : i0));
#pragma unroll
            for (u32 j = 0; j < 8; ++j) if (i0 + j * THREADS < n) f(i0 + j * THREADS, x[j]);
        }
    };
    bool missing = (w.force & kForceNoPosts) != 0;
    u32 polls = 0;
    if (tid < 256) sh.hist[tid] = 0;
    for (u32 i = tid; i < kListPosted / 32; i += THREADS) sh.owned[i] = 0;
    if (tid == 0) { sh.n = 0; sh.n_tie = 0; sh.kept = 0; sh.n_owned = 0; }
    __syncthreads();
    u64 prefix = 0;
    u32 top = 32 + shift, in = n, r = want;      // the r-th from the bottom among the `in` entries whose bits from `top` on are the prefix
    u32 width = top < 8 ? top : 8;
    auto count = [&](u64 e) { if ((e >> top) == prefix) atomicAdd(&sh.hist[static_cast<u32>(e >> (top - width)) & ((1u << width) - 1u)], 1u); };
    auto there = [&](u32 i, u64 x) {             // (at the first look, as a rule)
        while ((x & kPicked) == 0 && !missing) { __builtin_amdgcn_s_sleep(1); missing = ++polls > kPostPolls; x = ld_dev64(w.picked + i); }
        return entry(x);
    };
    if (in_lds) for (u32 i = tid; i < n && !missing; i += THREADS) sh.entry[i] = there(i, ld_dev64(w.picked + i));       // (one or two rounds, as a rule)
    else if (!missing) posted([&](u32 i, u64 x) { count(there(i, x)); });
    u32 range = 0;                               // of workgroup tid
    if (tid < walkers)
        while (((range = ld_dev(w.range + tid)) & kRangeKnown) == 0 && !missing) { __builtin_amdgcn_s_sleep(1); missing = ++polls > kPostPolls; }
    const bool any_missing = __any(missing);
    if ((tid & 63u) == 0) sh.missing[tid >> 6] = any_missing ? 1u : 0u;
    __syncthreads();
    u32 is_missing = 0;
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) is_missing |= sh.missing[i];
    if (is_missing != 0) {                       // uniform
        u64* const own = reinterpret_cast<u64*>(w.gidx);                 // where the indices of gathered entries otherwise are
        static_assert(2 * kListPosted <= kListGather, "room for them");
        if (tid < 256) sh.hist[tid] = 0;
        list_walk_own(w, rk, cnt, tid >> 6, THREADS / 64, [&](bool there, u32 key, u32 idx) {
            const u32 at = there && (key - win.lo) >> shift == bin ? atomicAdd(&sh.n, 1u) : n;             // n of them
            if (at < n) st_dev64(own + at, kPicked | (static_cast<u64>(key) << 32) | idx);
        });
        wait_dev();
        __syncthreads();
        if (tid == 0) sh.n = 0;
        from = own;
        if (in_lds) posted([&](u32 i, u64 x) { sh.entry[i] = entry(x); });
        else        posted([&](u32, u64 x) { count(entry(x)); });
        __syncthreads();
    }
    auto pick = [&]() {                          // the digit that the counts say
        if (tid < 64) {                          // four bins a lane, from the bottom
            const uint4 c4 = *reinterpret_cast<const uint4*>(sh.hist + 4 * tid);
            const u32 c[4] = {c4.x, c4.y, c4.z, c4.w}, sum = c[0] + c[1] + c[2] + c[3];
            u32 before = wave_incl_scan_u32(sum) - sum;
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
                if (before < r && r <= before + c[i]) { sh.bin = 4 * tid + i; sh.rem = r - before; sh.in = c[i]; }
                before += c[i];
            }
        }
        __syncthreads();
        prefix = (prefix << width) | sh.bin;
        r = sh.rem;
        in = sh.in;
        top -= width;
        width = top < 8 ? top : 8;
        if (tid < 256) sh.hist[tid] = 0;
        __syncthreads();
    };
    u32 held = n;                                // entries in LDS
    bool all_ties = true;                        // ... those that the threshold's equals are among
    if (!in_lds) {                               // only those that share its first digits are brought there
        pick();
        while (in > kListFound && top > 0) {     // uniform; (thousands of equal keys)
            posted([&](u32, u64 x) { count(entry(x)); });
            __syncthreads();
            pick();
        }
        all_ties = top >= 32;
        posted([&](u32, u64 x) { const u64 e = entry(x); if ((e >> top) == prefix) sh.entry[atomicAdd(&sh.n, 1u)] = e; });       // `in` of them
        __syncthreads();
        held = in;
        if (tid == 0) sh.n = 0;
        __syncthreads();
    }
    while (in > kShortPairs && top > 0) {        // uniform
        for (u32 i = tid; i < held; i += THREADS) count(sh.entry[i]);
        __syncthreads();
        pick();
    }
    for (u32 i = tid; i < held; i += THREADS)
        if ((sh.entry[i] >> top) == prefix) sh.pair[atomicAdd(&sh.n, 1u)] = sh.entry[i];       // `in` of them
    __syncthreads();
    if (tid < in) {
        const u64 mine = sh.pair[tid];
        u32 less = 0;
#pragma unroll 4
        for (u32 e = 0; e < in; ++e) less += sh.pair[e] < mine ? 1u : 0u;
        if (less + 1 == r) sh.found = mine;      // entries differ: one thread
    }
    __syncthreads();
    const u64 found = sh.found;
    const u32 T = top_key - static_cast<u32>(found >> 32), last = static_cast<u32>(found);
    if (tid < walkers && is_missing == 0) {
        const u64 was = __hip_atomic_exchange(w.verdict + tid, kPicked | (static_cast<u64>(T) << 32) | last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const u32 first = range & ((1u << kRangeBits) - 1u), number = (range & ~kRangeKnown) >> kRangeBits;
        if (was != kWalkerLeft && number != 0) {
            atomicAdd(&sh.n_owned, number);
            for (u32 i = first; i < first + number && i < kListPosted; ++i) atomicOr(&sh.owned[i / 32], 1u << (i % 32));
        }
    }
    auto tie = [&](u64 e) {
        if ((e >> 32) == (found >> 32)) {
            atomicAdd(&sh.n_tie, 1u);
            if (e <= found) atomicAdd(&sh.kept, 1u);
        }
    };
    if (all_ties) for (u32 i = tid; i < held; i += THREADS) tie(sh.entry[i]);
    else          posted([&](u32, u64 x) { tie(entry(x)); });
    __syncthreads();
    if (w.write && sh.n_owned != n) {            // uniform: some have left
        auto fix = [&](u32 i, u64 e) {
            if ((sh.owned[i / 32] >> (i % 32)) & 1u) return;
            const bool kept = e <= found;
            if (kept != (top_key - static_cast<u32>(e >> 32) >= win.mid)) list_fix_one<LC, PQ>(a, w, 0, static_cast<u32>(e), kept, nz);
        };
        for (u32 i = tid; i < n; i += THREADS) fix(i, in_lds ? sh.entry[i] : entry(ld_dev64(from + i)));
    }
    if (tid == 0) {
        Slot& slot = a.slots[0];
        u64 tie_end = slot.n;
        if (sh.kept < sh.n_tie) {
            const TensorDesc& td = a.td[a.chunk_map[last / kChunk]];
            tie_end = static_cast<u64>(last) - td.chunk_start * kChunk + (a.per_tensor ? 0 : td.flat_start) + 1;
        }
        slot.prefix = T; slot.remaining = sh.kept; slot.n_tie = sh.n_tie; slot.need_tie = 0; slot.tie_end = tie_end; slot.state = kDone;
        *results = select_record(slot, true, T, sh.kept, sh.n_tie, tie_end, is_missing == 0 ? slot.path : 3);
    }
}

// Every workgroup finds the bin of rank k - above from the counts.  Elements in the bins beside it are settled here:
// wrong decisions are queued in LDS, so that their chains of dependent loads run side by side.
// (Several rankings: an L-C step has one.)
__global__ __launch_bounds__(kBlock) void k_list_gather(DataArgs a, ListArgs w) {
    constexpr u32 kQueue = 2048;
    constexpr u32 kFound = 1024;
    __shared__ ListFindShared<kBlock> find;
    __shared__ u32 s_queue[kQueue];                        // wrong decisions: entry, top bit = the right one
    __shared__ u32 s_fkey[kFound], s_fidx[kFound];         // entries in the bin (one reservation per workgroup: updates of
                                                           // one counter that return a value take turns)
    __shared__ u32 s_n, s_f, s_base, s_max, s_maxc;
    const u32 s = blockIdx.x / w.parts, part = blockIdx.x % w.parts, tid = threadIdx.x, lane = tid & 63u;
    const ListRank rk = w.rank[s];
    const ListWin win = w.win[s];
    const Slot& slot = a.slots[s];
    if (part != 0 && part * (kBlock / 64) >= rk.n_segs) return;          // uniform
    const u32 k = static_cast<u32>(slot.k), n_all = static_cast<u32>(slot.n);
    const u32 state = slot.state;
    const ListFound f = list_find<kBlock>(w, find, s, rk, win, k);
    const bool crowded = win_crowded(win), ok = !crowded && f.want != 0 && f.n_in <= w.gather_cap;
    if (part == 0 && tid == 0) w.bin_want[s] = state == kSelecting && ok ? f.want : 0;
    if (state != kSelecting) return;                       // uniform; k == 0: nothing listed
    if (tid == 0) { s_n = 0; s_f = 0; s_max = 0; s_maxc = 0; }
    const u32 n_in = f.n_in, lo = win.lo, bin = f.bin, shift = win_shift(win), mid_bin = win_mid_bin(win);
    if (part == 0) {
        const u32 from = lo + (bin << shift), to = from + ((1u << shift) - 1u);
        if (crowded) {
            list_leave<kBlock>(a, w, s, lo, win.hi, k, 0, kStateUnsure);
        } else if (f.want == 0) {
            const ListState x = list_window_state(win, n_all, k, f.above, f.listed);
            list_leave<kBlock>(a, w, s, x.a, x.b, x.rank, x.n, 0);
        } else if (!ok || n_in > kListRanked) {
            list_leave<kBlock>(a, w, s, from, to < win.hi ? to : win.hi, f.want, n_in, ok ? kStateMaybe : 0);
        }
    }
    if (!ok) return;                                       // uniform over all workgroups of the ranking
    __syncthreads();
    const u32 g = s / a.J, j = s - g * a.J;
    int nz = 0;
    u32 most = 0, mostc = 0;
    // uniform.  Many: a walk over the list to count them first is cheaper than a reservation for every 64 (4 M weights widened
    // from 8 bits, 60 to 200 thousand ties: 25 us, 50 without); few: it is not (2 to 4 thousand of 20 M weights: 20 us, 31 with).
    const bool many = n_in > 8 * kFound;
    u32* gkey = w.gkey + static_cast<u64>(s) * w.gather_cap;
    u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
    const u32 first_seg = part * (kBlock / 64) + (tid >> 6), stride = w.parts * (kBlock / 64);
    auto settle_beside = [&](bool there, u32 key, u64 at, bool* found) {
        const u32 b = (key - lo) >> shift;
        const bool wrong = w.write && there && b != bin && (b > bin) != (b >= mid_bin);
        *found = there && b == bin;
        const u32 q = wave_push(&s_n, wrong);
        if (wrong) {
            if (q < kQueue) s_queue[q] = static_cast<u32>(at - rk.base) | (b > bin ? 0x80000000u : 0u);
            else            list_fix_one<false, false>(a, w, j, w.idx[at], b > bin, &nz);
        }
    };
    if (n_in <= kFound) {                                  // the buffer holds them wherever they are found
        list_walk(w, s, rk, first_seg, stride, find.cnt, [&](bool there, u32 key, u64 at) {
            bool found;
            settle_beside(there, key, at, &found);
            const u32 f = wave_push(&s_f, found);
            if (found) {
                s_fkey[f] = key;
                s_fidx[f] = static_cast<u32>(at - rk.base);
            }
        });
    } else {
        u32 next = 0;
        if (many) {                                        // one reservation for all that this wavefront will find
            list_walk(w, s, rk, first_seg, stride, find.cnt, [&](bool there, u32 key, u64) {
                next += static_cast<u32>(__popcll(__ballot(there && ((key - lo) >> shift) == bin)));
            });
            if (lane == 0 && next) next = atomicAdd(&w.gathered[static_cast<u64>(s) * kListLine], next);
            next = __shfl(next, 0, 64);
        }
        list_walk(w, s, rk, first_seg, stride, find.cnt, [&](bool there, u32 key, u64 at) {
            bool found;
            settle_beside(there, key, at, &found);
            if (found) {
                most = key > most ? key : most;
                mostc = ~key > mostc ? ~key : mostc;
            }
            const u32 f = many ? kFound : wave_push(&s_f, found);
            if (found && f < kFound) {
                s_fkey[f] = key;
                s_fidx[f] = static_cast<u32>(at - rk.base);
            }
            const u64 direct = __ballot(found && f >= kFound);           // straight to the list
            if (direct == 0) return;
            u32 to = next;
            if (!many) {
                const int leader = __ffsll(static_cast<long long>(direct)) - 1;
                if (static_cast<int>(lane) == leader) to = atomicAdd(&w.gathered[static_cast<u64>(s) * kListLine], static_cast<u32>(__popcll(direct)));
                to = __shfl(to, leader, 64);
            }
            next += static_cast<u32>(__popcll(direct));
            to += lanes_below(direct);
            if (((direct >> lane) & 1u) && to < w.gather_cap) { gkey[to] = key; gidx[to] = w.idx[at]; }
        });
    }
    if (n_in > kListRanked) {                              // are they all equal?
        atomicMax(&s_max, most);
        atomicMax(&s_maxc, mostc);
    }
    __syncthreads();
    const u32 n_f = s_f < kFound ? s_f : kFound, n_q = s_n < kQueue ? s_n : kQueue;
    if (tid == 0 && n_f) s_base = atomicAdd(&w.gathered[static_cast<u64>(s) * kListLine], n_f);
    if (tid == 0 && s_maxc) { atomicMax(&w.gmax[s], s_max); atomicMax(&w.gmaxc[s], s_maxc); }
    list_fix_queue<false, false, kBlock>(a, w, j, w.idx + rk.base, s_queue, n_q, &nz);
    __syncthreads();
    for (u32 f = tid; f < n_f; f += kBlock) {
        const u32 to = s_base + f;
        if (to < w.gather_cap) { gkey[to] = s_fkey[f]; gidx[to] = w.idx[rk.base + s_fidx[f]]; }
    }
}

// Wrong provisional decisions that a wavefront meets are queued in its own part of LDS, so that their chains of dependent loads run
// side by side afterwards.  They are the listed elements between the estimate's bin and the threshold's (without it): all
// kept where the estimate was too high, all dropped where it was too low.
template <u32 ROOM>
struct WaveQueue {
    u32* at;
    u32 n;                 // uniform
    bool keep;
    u32 lo, shift, bin, mid_bin;
    template <bool LC, bool PQ>
    __device__ inline bool offer(const DataArgs& a, const ListArgs& w, u32 j, bool there, u32 key, u32 idx, int* nz) {     // true: the entry is in the threshold's bin
        const u32 b = (key - lo) >> shift;
        const bool wrong = w.write && there && b != bin && (b > bin) != (b >= mid_bin);
        const u64 m = __ballot(wrong);
        if (m != 0) {                                      // uniform
            const u32 q = n + lanes_below(m);
            if (wrong) {
                if (q < ROOM) at[q] = idx;
                else          list_fix_one<LC, PQ>(a, w, j, idx, keep, nz);
            }
            n += static_cast<u32>(__popcll(m));
        }
        return there && b == bin;
    }
    template <bool LC, bool PQ>
    __device__ inline void fix(const DataArgs& a, const ListArgs& w, u32 j, int* nz) const {
        constexpr int B = 4;
        const u32 lane = threadIdx.x & 63u, upto = n < ROOM ? n : ROOM;
        for (u32 q0 = lane; q0 < upto; q0 += 64 * B) {
            u32 idx[B];
            bool to[B], on[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                on[b] = q0 + 64 * b < upto;
                idx[b] = on[b] ? at[q0 + 64 * b] : 0u;
                to[b] = keep;
            }
            list_fix<LC, PQ, B>(a, w, j, idx, to, on, nz);
        }
    }
};

// All entries of a long bin (ties, as a rule) to the ranking's gathered ones: one reservation for what a wavefront will find, which
// it counts first (4 M weights widened from 8 bits, 60 to 200 thousand ties: 25 us, 50 with a reservation for every 64).
// *most, *mostc: the largest key found and the complement of the smallest.
template <bool LC, bool PQ, u32 ROOM>
__device__ inline void list_gather_many(const DataArgs& a, const ListArgs& w, u32 s, u32 j, const ListRank& rk, const u32* cnt_of, u32 first_seg, u32 stride,
                                        WaveQueue<ROOM>& queue, u32* most, u32* mostc, int* nz) {
    const u32 lane = threadIdx.x & 63u;
    u32 next = 0;
    list_walk_own(w, rk, cnt_of, first_seg, stride, [&](bool there, u32 key, u32) {
        next += static_cast<u32>(__popcll(__ballot(there && ((key - queue.lo) >> queue.shift) == queue.bin)));
    });
    if (lane == 0 && next) next = add_dev(&w.gathered[static_cast<u64>(s) * kListLine], next);
    next = __shfl(next, 0, 64);
    u32* gkey = w.gkey + static_cast<u64>(s) * w.gather_cap;
    u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
    list_walk_own(w, rk, cnt_of, first_seg, stride, [&](bool there, u32 key, u32 idx) {
        const bool found = queue.template offer<LC, PQ>(a, w, j, there, key, idx, nz);
        const u64 m = __ballot(found);
        if (m == 0) return;                                // uniform
        const u32 to = next + lanes_below(m);
        if (found) {
            *most = key > *most ? key : *most;
            *mostc = ~key > *mostc ? ~key : *mostc;
            if (to < w.gather_cap) { st_dev(gkey + to, key); st_dev(gidx + to, idx); }
        }
        next += static_cast<u32>(__popcll(m));
    });
}

// Where a ranking goes that its list does not settle: to list_fallback, by one workgroup.  True: the gathered entries will be ranked
// there or in list_rank, so they have to be gathered.
template <int THREADS>
__device__ inline bool list_leave_open(const DataArgs& a, const ListArgs& w, u32 s, const ListWin& win, const ListFound& f, u32 n, u32 k, bool leave) {
    const u32 from = win.lo + (f.bin << win_shift(win)), to = from + ((1u << win_shift(win)) - 1u);
    const bool fits = f.n_in <= w.gather_cap;
    if (leave) {
        if (f.want == 0) {
            const ListState x = list_window_state(win, n, k, f.above, f.listed);
            list_leave<THREADS>(a, w, s, x.a, x.b, x.rank, x.n, 0);
        } else {
            list_leave<THREADS>(a, w, s, from, to < win.hi ? to : win.hi, f.want, f.n_in, fits ? kStateMaybe : 0);
        }
    }
    return f.want != 0 && fits;
}

// ---- what the lists leave open ----------------------------------------------------------------------------------
//
// Rankings whose threshold is not in their list (the window missed it, the list is full), whose window is crowded, or whose
// threshold has more ties than one workgroup should rank: counts of the keys in an interval (one read of the population), the
// bin that becomes the next interval until it is a single key, ties per chunk (another read), the tie rule, and the outputs (a
// third read, or the ties alone where everything else is right).

// A chunk's elements, kPer per thread, and their keys: 0xFFFFFFFF past the tensor's end (above every interval and equal to no
// threshold).
template <bool LC, bool VEC, int THREADS>
struct ChunkKeys {
    static constexpr int kQuads = kChunk / (4 * THREADS), kPer = 4 * kQuads;
    float v[kQuads][4], l[LC ? kQuads : 1][4];
    u32 there;
    float mu;
    // The loads.  Those of a whole chunk stay in flight (their number is the same for every lane, so whoever needs older ones
    // need not wait for these); a ragged one waits for its own.
    __device__ inline void fetch(const DataArgs& a, u64 c) {
        const TensorDesc& td = a.td[a.chunk_map[c]];
        const u64 base = (c - td.chunk_start) * kChunk, n = td.n;
        mu = a.mu;
        if (VEC && base + kChunk <= n) {                   // uniform
            there = 0xFFFFFFFFu;
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                const u64 e0 = base + static_cast<u64>(q) * (4 * THREADS) + threadIdx.x * 4;
                const float4 x = *reinterpret_cast<const float4*>(td.w + e0);
                v[q][0] = x.x; v[q][1] = x.y; v[q][2] = x.z; v[q][3] = x.w;
                if (LC) {
                    const float4 y = *reinterpret_cast<const float4*>(td.lam + e0);
                    l[q][0] = y.x; l[q][1] = y.y; l[q][2] = y.z; l[q][3] = y.w;
                }
            }
            return;
        }
        there = 0;
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            const u64 e0 = base + static_cast<u64>(q) * (4 * THREADS) + threadIdx.x * 4;
            if (e0 < n) {
                load4<VEC>(td.w, e0, n, v[q]);
                if (LC) load4<VEC>(td.lam, e0, n, l[q]);
                there |= ((1u << (n - e0 < 4 ? static_cast<u32>(n - e0) : 4u)) - 1u) << (4 * q);
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
    }
    __device__ inline u32 key(int e) const {
        const float x = LC ? lc_shift(v[e / 4][e % 4], l[LC ? e / 4 : 0][e % 4], mu) : v[e / 4][e % 4];
        return (there >> e) & 1u ? mag_key(x) : 0xFFFFFFFFu;
    }
    // words: B counts, B largest distances from lo (plus one), B smallest ones (their complements)
    __device__ inline void count(u32* words, u32 B, u32 lo, u32 span, u32 shift) const {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const u32 d = key(e) - lo, b = d >> shift;
            const bool in = d <= span;
            const u64 all = __ballot(in);
            if (all == 0) continue;                        // uniform
            bool mine = in;
            if (__popcll(all) > 12) {                      // lanes that meet on a counter take turns: ties are added up first
                const int leader = __ffsll(static_cast<long long>(all)) - 1;
                const u32 d0 = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(d), leader));
                const u64 same = __ballot(in && d == d0);
                if (static_cast<int>(threadIdx.x & 63u) == leader) atomicAdd(&words[b], static_cast<u32>(__popcll(same)) - 1u);
                mine = in && (d != d0 || static_cast<int>(threadIdx.x & 63u) == leader);
            }
            if (mine) {
                atomicAdd(&words[b], 1u);
                if (words[B + b] < d + 1u) atomicMax(&words[B + b], d + 1u);           // seldom: a plain look first
                if (words[2 * B + b] < ~d) atomicMax(&words[2 * B + b], ~d);
            }
        }
    }
    // The same for several intervals at once, a[j] .. a[j] + span[j]: tab[leading 11 bits of a key] are those (a bit each) that
    // hold keys of that kind, so that a key costs a look-up and its own intervals.
    __device__ inline void count_many(u32* words, u32 B, const u16* tab, const u32* a, const u32* span, const u32* shift) const {
        const u32 lane = threadIdx.x & 63u;
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const u32 x = key(e);
            u32 of = x <= 0x7FFFFFFFu ? tab[x >> 20] : 0u;
            const u64 all = __ballot(of != 0);
            if (all == 0) continue;                        // uniform
            const int leader = __ffsll(static_cast<long long>(all)) - 1;
            const u32 x0 = static_cast<u32>(__builtin_amdgcn_readlane(static_cast<int>(x), leader));
            const u64 same = __ballot(x == x0);
            u32 n = 1;
            if (__popcll(same) > 12) {                     // ties are added up first
                n = static_cast<int>(lane) == leader ? static_cast<u32>(__popcll(same)) : 1u;
                if (x == x0 && static_cast<int>(lane) != leader) of = 0;
            }
            while (of) {
                const u32 j = static_cast<u32>(__ffs(of)) - 1u, d = x - a[j];
                of &= of - 1u;
                if (d > span[j]) continue;
                u32* to = words + j * 3 * B + (d >> (shift[j] & 0xFFu));
                atomicAdd(to, n);
                if (to[B] < d + 1u) atomicMax(to + B, d + 1u);
                if (to[2 * B] < ~d) atomicMax(to + 2 * B, ~d);
            }
        }
    }
    // The outputs of chunk c for the rankings in `rankings` (L-C step: the one), whose thresholds are T and ends of kept ties `end`;
    // adds this thread's non-zero codes to *nz.
    template <bool PQ>
    __device__ inline void apply(const DataArgs& a, const OutDesc* out, u64 c, u32 rankings, const u32* T, const u64* end, bool vec, u32* nz) const {
        const u32 t = a.chunk_map[c];
        const TensorDesc& td = a.td[t];
        const u64 base = (c - td.chunk_start) * kChunk, n = td.n, idx0 = a.per_tensor ? 0 : td.flat_start;
        vec = vec && VEC;
        for (u32 js = rankings; js != 0; js &= js - 1u) {  // uniform
            const u32 j = static_cast<u32>(__ffs(js)) - 1u, Tj = T[j];
            const u64 endj = end[j];
            const OutDesc o = out[static_cast<u64>(j) * a.n_tensors + t];
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                const u64 e0 = base + static_cast<u64>(q) * (4 * THREADS) + threadIdx.x * 4;
                if (e0 >= n) continue;
                float th[4], ln[4], gr[4];
                u8 m[4];
                u16 h[4] = {0, 0, 0, 0};
                if constexpr (LC) {
                    lc_update4<PQ>(v[q], l[q], a.mu, Tj, idx0 + e0, endj, th, ln, gr, m, h);
                    if (PQ)
                        for (int k = 0; k < 4; ++k) *nz += (e0 + k < n) && (h[k] & 0x7FFFu) != 0 ? 1u : 0u;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        m[k] = keep_rule(key(4 * q + k), Tj, idx0 + e0 + k, endj) ? 1 : 0;
                        th[k] = m[k] ? v[q][k] : 0.0f;
                    }
                    if (o.theta16)
                        for (int k = 0; k < 4; ++k) h[k] = f32_to_f16_rne(th[k]);
                }
                if (vec && e0 + 4 <= n) {
                    if (o.theta) st4_stream(o.theta + e0, th[0], th[1], th[2], th[3]);
                    if ((!LC || PQ) && o.theta16) st_code4_stream(o.theta16 + e0, h[0], h[1], h[2], h[3]);
                    if (LC) st4_stream(td.lam_out + e0, ln[0], ln[1], ln[2], ln[3]);
                    if (LC && td.grad) st4_stream(td.grad + e0, gr[0], gr[1], gr[2], gr[3]);
                    if (o.mask) st_mask4_stream(o.mask + e0, m[0], m[1], m[2], m[3]);
                } else {
                    if (o.theta) store4<false>(o.theta, e0, n, th);
                    if ((!LC || PQ) && o.theta16) store4_u16<false>(o.theta16, e0, n, h);
                    if (LC) store4<false>(td.lam_out, e0, n, ln);
                    if (LC && td.grad) store4<false>(td.grad, e0, n, gr);
                    if (o.mask) store4_u8<false>(o.mask, e0, n, m);
                }
            }
        }
    }
    __device__ inline u32 above(u32 hi) const {            // of the wavefront
        u32 n = 0;
#pragma unroll
        for (int e = 0; e < kPer; ++e) n += static_cast<u32>(__popcll(__ballot(key(e) - hi - 1u < 0x7FFFFFFFu - hi)));
        return n;
    }
    __device__ inline u32 equal(u32 T) const {             // of the wavefront
        u32 n = 0;
#pragma unroll
        for (int e = 0; e < kPer; ++e) n += static_cast<u32>(__popcll(__ballot(key(e) == T)));
        return n;
    }
};
// f(c, chunk) for the chunks c0 .. c1 that `want` asks for, until it returns true; the next one's loads are in flight meanwhile.
template <bool LC, bool VEC, int THREADS, typename Want, typename F>
__device__ inline void for_chunks(const DataArgs& a, u64 c0, u64 c1, Want&& want, F&& f) {
    ChunkKeys<LC, VEC, THREADS> x;
    auto next = [&](u64 c) { while (c < c1 && !want(c)) ++c; return c; };
    u64 c = next(c0);
    if constexpr (LC) {                                    // (two chunks of two arrays do not fit the registers)
        for (; c < c1; c = next(c + 1)) {
            x.fetch(a, c);
            if (f(c, x)) return;
        }
    } else {
        ChunkKeys<LC, VEC, THREADS> y;
        if (c < c1) x.fetch(a, c);
        while (c < c1) {                                   // uniform
            const u64 d = next(c + 1);
            if (d < c1) y.fetch(a, d);
            if (f(c, x)) return;
            if (d >= c1) return;
            c = next(d + 1);
            if (c < c1) x.fetch(a, c);
            if (f(d, y)) return;
        }
    }
}

__device__ inline u32 bins_shift(u32 span, u32 bins) {     // (d >> shift) < bins for every d <= span
    const u32 bits = 32u - static_cast<u32>(__builtin_clz(span | 1u)), have = 31u - static_cast<u32>(__builtin_clz(bins));
    return bits > have ? bits - have : 0u;
}

// The next interval, from the keys that lie in the bin of the rank: word(b) keys in bin b of B over st's interval, word(B + b) and
// word(2 B + b) their range (as ChunkKeys::count leaves them), `above` keys above the interval (needed when it is unsure).
// All threads; pick: three words of LDS.  Ends with a barrier, after the last use of the words.
template <int THREADS, typename Word>
__device__ inline ListState next_interval(const ListState& st, u32 B, u32 above, u32 n_all, u32* s_wave, u32* pick, Word&& word) {
    const u32 per = (B + THREADS - 1) / THREADS, first = threadIdx.x * per;            // this thread's bins, from the top
    u32 sum = 0, all;
    for (u32 i = first; i < first + per && i < B; ++i) sum += word(B - 1 - i);
    if (threadIdx.x < 3) pick[threadIdx.x] = 0;
    u32 before = wg_incl_scan_u32<THREADS>(sum, s_wave, &all) - sum;
    const bool unsure = (st.flags & kStateUnsure) != 0;
    const bool inside = !unsure || (above < st.rank && st.rank - above <= all);
    const u32 rank = unsure ? st.rank - above : st.rank;
    if (inside)
        for (u32 i = first; i < first + per && i < B; ++i) {
            const u32 v = word(B - 1 - i);
            if (before < rank && rank <= before + v) { pick[0] = B - 1 - i; pick[1] = rank - before; pick[2] = v; }
            before += v;
        }
    __syncthreads();
    ListState x{};
    if (inside) {
        x.a = st.a + ~word(2 * B + pick[0]);
        x.b = st.a + word(B + pick[0]) - 1u;
        x.rank = pick[1];
        x.n = pick[2];
    } else if (above >= st.rank) {
        x.a = st.b + 1u; x.b = 0x7FFFFFFFu; x.rank = st.rank; x.n = above;
    } else {
        x.a = 0; x.b = st.a - 1u; x.rank = st.rank - above - all; x.n = n_all - above - all;
    }
    __syncthreads();
    return x;
}

constexpr u32 kFallbackWords = 3 * 4096;         // histograms of one population's rankings in LDS

// One ranking by one workgroup (k_list_finish): `st` says where its threshold is, `nz` are this thread's corrections so far of
// the count of non-zero codes.
template <bool LC, bool VEC, bool PQ>
__device__ inline void list_alone(const DataArgs& a, const ListArgs& w, u32* words, u32* s_wave, u32* s_pick, u64* s_end, u32 s, ListState st, int nz,
                                  condensa_select* results, int n_groups, int vec_out) {
    constexpr int THREADS = kListThreads;
    const u32 tid = threadIdx.x, lane = tid & 63u, g = s / a.J, j = s - g * a.J;
    Slot& slot = a.slots[s];
    const u64 cb = a.per_tensor ? a.td[g].chunk_start : 0, ce = a.per_tensor ? a.td[g + 1].chunk_start : a.n_chunks;
    const bool tied = (st.flags & kStateTied) != 0;
    auto any = [](u64) { return true; };
    constexpr u32 B = kFallbackWords / 3;
    for (int level = 0; level < kFallbackLevels && (st.a < st.b || (st.flags & kStateUnsure)); ++level) {
        for (u32 i = tid; i < kFallbackWords; i += THREADS) words[i] = 0;
        if (tid == 0) s_pick[3] = 0;
        __syncthreads();
        const u32 span = st.b - st.a, shift = bins_shift(span, B);
        for_chunks<LC, VEC, THREADS>(a, cb, ce, any, [&](u64, const auto& ck) {
            ck.count(words, B, st.a, span, shift);
            if (!(st.flags & kStateUnsure)) return false;  // uniform
            const u32 above = ck.above(st.b);
            if (lane == 0 && above) atomicAdd(&s_pick[3], above);
            return false;
        });
        __syncthreads();
        st = next_interval<THREADS>(st, B, s_pick[3], static_cast<u32>(slot.n), s_wave, s_pick, [&](u32 i) { return words[i]; });
    }
    const u32 T = st.a;
    u32 last = 0xFFFFFFFFu;
    u64 tie_end = slot.n;
    if (st.rank < st.n) {                                  // uniform: the chunk, then the element that ends the kept ties
        u32 cum = 0;
        for_chunks<LC, VEC, THREADS>(a, cb, ce, any, [&](u64 c, const auto& ck) {
#pragma unroll
            for (int q = 0; q < ck.kQuads; ++q) {          // elements ascend with q, then the thread, then k
                u32 eq = 0, total;
#pragma unroll
                for (int k = 0; k < 4; ++k) eq |= ck.key(4 * q + k) == T ? 1u << k : 0u;
                const u32 mine = static_cast<u32>(__popc(eq)), upto = cum + wg_incl_scan_u32<THREADS>(mine, s_wave, &total);
                if (upto - mine < st.rank && st.rank <= upto) {
                    for (u32 skip = st.rank - (upto - mine) - 1; skip > 0; --skip) eq &= eq - 1;
                    s_pick[0] = q * (4 * THREADS) + tid * 4 + static_cast<u32>(__ffs(eq)) - 1u;
                }
                cum += total;
                if (cum < st.rank) continue;               // uniform
                __syncthreads();
                const TensorDesc& td = a.td[a.chunk_map[c]];
                last = static_cast<u32>(c) * kChunk + s_pick[0];
                tie_end = (c - td.chunk_start) * kChunk + s_pick[0] + (a.per_tensor ? 0 : td.flat_start) + 1;
                return true;
            }
            return false;
        });
        __syncthreads();
    }
    if (tid == 0) {
        slot.prefix = T; slot.remaining = st.rank; slot.n_tie = st.n; slot.need_tie = 0; slot.tie_end = tie_end; slot.state = kDone;
        results[static_cast<u64>(j) * n_groups + g] = select_record(slot, true, T, st.rank, st.n, tie_end, tied ? slot.path : 3);
    }
    if (!w.write) return;
    u32 codes = 0;
    if (tied) {                                            // the ties alone
        const bool kept = T >= w.win[s].mid;
        const u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
        constexpr int kB = 4;
        for (u32 i0 = tid; i0 < st.n; i0 += THREADS * kB) {
            u32 idx[kB];
            bool keep[kB], on[kB];
#pragma unroll
            for (int b = 0; b < kB; ++b) {
                const u32 i = i0 + b * THREADS;
                idx[b] = i < st.n ? gidx[i] : 0u;
                keep[b] = idx[b] <= last;
                on[b] = i < st.n && keep[b] != kept;
            }
            list_fix<LC, PQ, kB>(a, w, j, idx, keep, on, &nz);
        }
    } else {
        if (tid == 0) { s_pick[j] = T; s_end[j] = tie_end; }
        __syncthreads();
        for_chunks<LC, VEC, THREADS>(a, cb, ce, any, [&](u64 c, const auto& ck) {
            ck.template apply<PQ>(a, w.out, c, 1u << j, s_pick, s_end, vec_out != 0, &codes);
            return false;
        });
    }
    if (PQ && w.nnz_out) {                                 // modulo 2^32: the sums themselves are smaller
        u32 v = tied ? static_cast<u32>(nz) : codes, total;
        if (tied) for (u32 i = tid; i < static_cast<u32>(kListSegs); i += THREADS) v += w.nnz[i];
        __syncthreads();
        wg_incl_scan_u32<THREADS>(v, s_wave, &total);
        if (tid == 0) *w.nnz_out = total;
    }
}

// Rankings of populations of at most list_lone elements: one workgroup each does the counting, the gathering and the
// ranking on its list, and what that leaves open (65 536 weights, nine tenths zeros: 83-92 us the call, 317-358 when elements
// were ranked and written one at a time).
template <bool LC, bool VEC, bool PQ>
__global__ __launch_bounds__(kListThreads) void k_list_finish(DataArgs a, ListArgs w, condensa_select* results, int n_groups, int vec_out) {
    constexpr u32 kQueue = 4096;
    __shared__ ListShared sh;
    __shared__ __align__(8) u32 s_big[kFallbackWords];             // queue of wrong decisions; list_alone's histogram
    __shared__ u32 s_n, s_f, s_over, s_max, s_maxc, s_pick[kMaxJ];
    __shared__ u64 s_end[kMaxJ];
    const u32 tid = threadIdx.x, wave = tid >> 6;
    constexpr u32 kWaves = kListThreads / 64;
    const u32 s = blockIdx.x;
    const ListRank rk = w.rank[s];
    const ListWin win = w.win[s];
    const u32 g = s / a.J, j = s - g * a.J;
    Slot& slot = a.slots[s];
    int nz = 0;
    u32 want = 0, n = 0;
    bool in_lds = false, left = false;
    ListState st{};
    if (slot.state == kSelecting && win_crowded(win)) {    // uniform
        left = true;
        st.a = win.lo; st.b = win.hi; st.rank = static_cast<u32>(slot.k); st.flags = kStateUnsure;
    } else if (slot.state == kSelecting) {
        const u64 cw = tid < rk.n_segs ? w.cnt[static_cast<u64>(s) * w.max_segs + tid] : 0;       // n_segs <= kListSegs == kListThreads
        const u32 k = static_cast<u32>(slot.k);
        if (tid < static_cast<u32>(kListBins)) sh.hist[tid] = 0;
        if (tid == 0) { s_n = 0; s_f = 0; s_over = 0; s_max = 0; s_maxc = 0; }
        __syncthreads();
        if (static_cast<u32>(cw) > rk.seg_cap) s_over = 1;
        u32 above, listed;
        wg_incl_scan_u32<kListThreads>(static_cast<u32>(cw >> 32), sh.wave, &above);
        wg_incl_scan_u32<kListThreads>(static_cast<u32>(cw), sh.wave, &listed);
        const u32 lo = win.lo, shift = win_shift(win), mid_bin = win_mid_bin(win);
        if (s_over != 0 || above >= k || k - above > listed) {           // uniform
            left = true;
            st = list_window_state(win, static_cast<u32>(slot.n), k, above, listed);
        } else {
            list_walk(w, s, rk, wave, kWaves, nullptr, [&](bool there, u32 key, u64) { wave_count(sh.hist, there, there ? (key - lo) >> shift : 0u); });
            __syncthreads();
            u32 bin;
            list_pick(sh, true, k - above, &bin, &want, &n);
            if (n > w.gather_cap) {
                left = true;
                st.a = lo + (bin << shift); st.b = st.a + ((1u << shift) - 1u); st.rank = want; st.n = n;
                st.b = st.b < win.hi ? st.b : win.hi;
            } else {
                u32* gkey = w.gkey + static_cast<u64>(s) * w.gather_cap;
                u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
                const u32* __restrict__ ids = w.idx + rk.base;
                in_lds = n <= kListRanked;
                u32 most = 0, mostc = 0;
                list_walk(w, s, rk, wave, kWaves, nullptr, [&](bool there, u32 key, u64 at) {
                    const u32 b = (key - lo) >> shift, entry = static_cast<u32>(at - rk.base);
                    const bool found = there && b == bin, wrong = w.write && there && b != bin && (b > bin) != (b >= mid_bin);
                    const u32 f = wave_push(&s_f, found);  // n of them; their indices are fetched below, side by side
                    if (found) {
                        most = key > most ? key : most;
                        mostc = ~key > mostc ? ~key : mostc;
                        if (in_lds) { sh.key[f] = key; sh.idx[f] = entry; }
                        else        { gkey[f] = key; gidx[f] = entry; }
                    }
                    const u32 q = wave_push(&s_n, wrong);
                    if (wrong) {
                        if (q < kQueue) s_big[q] = entry | (b > bin ? 0x80000000u : 0u);
                        else            list_fix_one<LC, PQ>(a, w, j, ids[entry], b > bin, &nz);
                    }
                });
                if (!in_lds) { atomicMax(&s_max, most); atomicMax(&s_maxc, mostc); }
                __syncthreads();
                if (in_lds) for (u32 f = tid; f < n; f += kListThreads) sh.idx[f] = ids[sh.idx[f]];
                else        for (u32 f = tid; f < n; f += kListThreads) gidx[f] = ids[gidx[f]];
                list_fix_queue<LC, PQ, kListThreads>(a, w, j, ids, s_big, s_n < kQueue ? s_n : kQueue, &nz);
                __threadfence_block();                     // the gathered entries are read by other threads below
                __syncthreads();
                if (!in_lds && s_max == ~s_maxc) {         // uniform: thousands of ties
                    left = true;
                    st.a = st.b = s_max; st.rank = want; st.n = n; st.flags = kStateTied;
                }
            }
        }
    }
    if (left) list_alone<LC, VEC, PQ>(a, w, s_big, sh.wave, s_pick, s_end, s, st, nz, results, n_groups, vec_out);
    else      list_rank<LC, PQ, kListThreads, false>(a, w, sh, s, want, n, in_lds, nz, 0, 1, results, n_groups);
}

// ---- the whole grid on what the lists leave open -------------------------------------------------------------------
//
// All rankings of a call that are left open go through the phases together, however many there are.  A workgroup that takes
// part takes the same share of every phase, and all of them meet between two phases.  For that they must all be running:
// each one registers, and when all have, or some time has passed, the first one closes the register and tells those in it
// how many they are.  Who comes too late leaves.  So nobody ever waits for a workgroup that is not running.
// A register, a counter or a flag that hundreds of workgroups update or poll costs some 0.1 us for each of them, so there are
// kMeetGroups of each, in cache lines of their own.
// What one phase hands to the next goes through device-scope loads, stores and atomics alone (ld_dev and its like), which
// pass the caches of compute units and dies; waiting for them (s_waitcnt) before the workgroup counts as arrived is all they
// need.  A fence of device scope would write back and invalidate a die's whole cache: with one per wavefront a phase took 100 us.
constexpr u32 kMeetGroups = 16, kMeetLine = 32;  // words of a 128-byte line
constexpr u32 kMeetClosed = 0x80000000u;
constexpr u32 kMeetWords = (3 * kMeetGroups + 2) * kMeetLine;
struct Meet {
    u32* word;
    u32 rank, size, met;       // this workgroup's number, how many take part, meetings so far
    __device__ inline u32* joined(u32 g) const { return word + g * kMeetLine; }                            // registered | kMeetClosed
    __device__ inline u32* arrived(u32 g) const { return word + (kMeetGroups + g) * kMeetLine; }
    __device__ inline u32* told(u32 g) const { return word + (2 * kMeetGroups + g) * kMeetLine; }          // [0] meetings over, [1] first number | kMeetClosed, [2] size
    __device__ inline u32* root(u32 i) const { return word + (3 * kMeetGroups + i) * kMeetLine; }          // 0: who is first, 1: groups arrived
};
// All threads; false: too late.  sh: three words of LDS.
__device__ inline bool meet_join(Meet& m, u32* words, u32* sh) {
    m.word = words;
    m.met = 0;
    const u32 tid = threadIdx.x;
    if (tid < 64) {
        const u32 g = blockIdx.x % kMeetGroups;
        u32 mine = 0, first = 0;
        if (tid == 0) {
            mine = add_dev(m.joined(g), 1u);
            first = mine == 0 && add_dev(m.root(0), 1u) == 0 ? 1u : 0u;
        }
        mine = __shfl(mine, 0, 64);
        first = __shfl(first, 0, 64);
        if (first) {                                       // wavefront 0 of the workgroup that was first: lane g minds group g
            for (int polls = 0; polls < 200; ++polls) {    // some 100 us at most
                u32 here = tid < kMeetGroups ? ld_dev(m.joined(tid)) : 0u;
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) here += __shfl_xor(here, d, 64);
                if (here == gridDim.x) break;
                __builtin_amdgcn_s_sleep(4);
            }
            u32 n = 0;
            if (tid < kMeetGroups) n = __hip_atomic_fetch_or(m.joined(tid), kMeetClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            u32 upto = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) { const u32 o = __shfl_up(upto, d, 64); if (static_cast<int>(tid) >= d) upto += o; }
            const u32 all = __shfl(upto, 63, 64);
            if (tid < kMeetGroups) {
                st_dev(m.told(tid) + 2, all);
                wait_dev();                                // the size is there before the flag
                st_dev(m.told(tid) + 1, (upto - n) | kMeetClosed);
            }
        }
        if (tid == 0) {
            sh[0] = 0;
            if (!(mine & kMeetClosed)) {                   // registered in time: the first one is running and will say so
                u32 from;
                while (((from = ld_dev(m.told(g) + 1)) & kMeetClosed) == 0) __builtin_amdgcn_s_sleep(2);
                wait_dev();
                sh[0] = 1;
                sh[1] = (from & ~kMeetClosed) + mine;
                sh[2] = ld_dev(m.told(g) + 2);
            }
        }
    }
    __syncthreads();
    const bool in = sh[0] != 0;
    m.rank = sh[1];
    m.size = sh[2];
    __syncthreads();
    return in;
}
// All threads of all workgroups that joined.
__device__ inline void meet(Meet& m) {
    wait_dev();                                            // every thread's stores have reached the device
    __syncthreads();
    ++m.met;
    if (threadIdx.x == 0) {
        const u32 g = m.rank % kMeetGroups, groups = m.size < kMeetGroups ? m.size : kMeetGroups;
        const u32 in_group = (m.size - g + kMeetGroups - 1) / kMeetGroups;
        bool over = false;
        if (add_dev(m.arrived(g), 1u) + 1 == in_group * m.met) over = add_dev(m.root(1), 1u) + 1 == groups * m.met;
        if (over) for (u32 i = 0; i < groups; ++i) st_dev(m.told(i), m.met);
        else      while (ld_dev(m.told(g)) < m.met) __builtin_amdgcn_s_sleep(2);
    }
    __syncthreads();
}

struct FallbackShared {
    u64 end[kMaxJ];
    u32 a[kMaxJ], span[kMaxJ], shift[kMaxJ], count[kMaxJ];
    u32 wave[kListThreads / 64];
    u32 pick[4];
    u16 tab[2048];
};

// Gathered entries that are many and all equal are ties (whose number and rank are known): list_fallback takes them.
__device__ inline bool list_tied(const ListArgs& w, u32 s) {
    return ld_dev(w.bin_want + s) != 0 && ld_dev(&w.gathered[static_cast<u64>(s) * kListLine]) > kListRanked && ld_dev(w.gmax + s) == ~ld_dev(w.gmaxc + s);
}
// State of a special ranking; false: list_rank takes it.
__device__ inline bool list_state(const ListArgs& w, u32 s, ListState* st) {
    *st = ld_state(w.state + s);
    if (!(st->flags & kStateMaybe)) return true;
    if (!list_tied(w, s)) return false;
    st->a = st->b = ld_dev(w.gmax + s);
    st->n = ld_dev(&w.gathered[static_cast<u64>(s) * kListLine]);
    st->flags = kStateTied;
    return true;
}

// Long lists: gathered ties are counted by chunk from where they lie, not by another sweep over the weights (604 M weights in binary16, 190 thousand ties, L-C step 2 855 ->
// 2 010 us; 302 M 1 490 -> 1 055), unless so many meet in a chunk that their updates take turns (4.7 M weights in E4M3, hundreds in a chunk: 212 us swept, 295 so).
__device__ inline bool list_ties_counted(const DataArgs& a, const ListState& st) { return (st.flags & kStateTied) && st.n <= 16 * a.n_chunks; }

// `words`: kFallbackWords of LDS.  `tied`: some suspected ties are ties; `search`: some of those have to be searched.
template <bool LC, bool VEC, bool PQ, bool LONG, int THREADS>
__device__ inline void list_fallback(const DataArgs& a, const ListArgs& w, Meet& m, FallbackShared& sh, u32* words, condensa_select* results, int n_groups,
                                     int vec_out, bool tied, bool search) {
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 n_special = ld_dev(&w.fb->special), B = w.fb_bins, n_apply = ld_dev(&w.fb->apply);       // final: counted before the last meeting
    const u64 c0 = a.n_chunks * m.rank / m.size, c1 = a.n_chunks * (m.rank + 1) / m.size;      // this workgroup's chunks
    auto group_of = [&](u64 c) { return a.per_tensor ? a.chunk_map[c] : 0u; };
    // the rankings (a bit each) of chunk c's population in one of the masks, looked up where the population changes
    u32 seen = 0xFFFFFFFFu, seen_mask = 0;
    auto wanted = [&](const u32* masks) {
        seen = 0xFFFFFFFFu;
        return [&, masks](u64 c) {
            const u32 g = group_of(c);
            if (g != seen) { seen = g; seen_mask = ld_dev(masks + g); }
            return seen_mask != 0;
        };
    };

    for (int level = 0; level < kFallbackLevels && ld_dev(&w.fb->open[level]) != 0; ++level) {
        // ---- counts of the keys in the intervals
        u32 cur = 0xFFFFFFFFu, mask = 0, unsure = 0;
        bool several = false;                              // the leading digits of the keys say whose they can be
        auto flush = [&]() {
            __syncthreads();
            for (u32 js = mask; js != 0; js &= js - 1u) {
                const u32 j = static_cast<u32>(__ffs(js)) - 1u;
                const u64 s = static_cast<u64>(cur) * a.J + j;
                const u32* from = words + j * 3 * B;
                u32* to = w.fb_hist + s * 3 * B;
                for (u32 i = tid; i < B; i += THREADS) {
                    if (from[i] == 0) continue;
                    add_dev(&to[i], from[i]);
                    max_dev(&to[B + i], from[B + i]);
                    max_dev(&to[2 * B + i], from[2 * B + i]);
                }
                if (tid == 0 && sh.count[j]) add_dev(&w.fb_above[s], sh.count[j]);
            }
            __syncthreads();
        };
        for_chunks<LC, VEC, THREADS>(a, c0, c1, wanted(w.open_of), [&](u64 c, const auto& ck) {
            const u32 g = group_of(c);
            if (g != cur) {                                // uniform
                if (mask) flush();
                cur = g;
                mask = ld_dev(&w.open_of[g]);
                unsure = 0;
                for (u32 i = tid; i < 3 * B * static_cast<u32>(a.J); i += THREADS) words[i] = 0;
                if (tid < static_cast<u32>(a.J)) {
                    const ListState st = ld_state(w.state + static_cast<u64>(g) * a.J + tid);
                    sh.a[tid] = st.a;
                    sh.span[tid] = st.b - st.a;
                    sh.shift[tid] = bins_shift(st.b - st.a, B) | (st.flags & kStateUnsure ? 0x100u : 0u);
                    sh.count[tid] = 0;
                }
                __syncthreads();
                for (u32 j = 0; j < static_cast<u32>(a.J); ++j) unsure |= sh.shift[j] & 0x100u ? 1u << j : 0u;
                several = __popc(mask) > 2;
                if (several) {
                    for (u32 i = tid; i < 2048; i += THREADS) {
                        u32 of = 0;
                        for (u32 js = mask; js != 0; js &= js - 1u) {
                            const u32 j = static_cast<u32>(__ffs(js)) - 1u;
                            if (i >= sh.a[j] >> 20 && i <= (sh.a[j] + sh.span[j]) >> 20) of |= 1u << j;
                        }
                        sh.tab[i] = static_cast<u16>(of);
                    }
                    __syncthreads();
                }
            }
            if (several) ck.count_many(words, B, sh.tab, sh.a, sh.span, sh.shift);
            for (u32 js = several ? unsure & mask : mask; js != 0; js &= js - 1u) {            // uniform
                const u32 j = static_cast<u32>(__ffs(js)) - 1u;
                if (!several) ck.count(words + j * 3 * B, B, sh.a[j], sh.span[j], sh.shift[j] & 0xFFu);
                if (!((unsure >> j) & 1u)) continue;
                const u32 above = ck.above(sh.a[j] + sh.span[j]);
                if (lane == 0 && above) atomicAdd(&sh.count[j], above);
            }
            return false;
        });
        if (mask) flush();
        meet(m);
        // ---- the next intervals
        for (u32 f = m.rank; f < n_special; f += m.size) {
            const u32 s = ld_dev(w.special + f), g = s / a.J, j = s - g * a.J;
            if (((ld_dev(&w.open_of[g]) >> j) & 1u) == 0) continue;      // uniform: this bit is this workgroup's to change
            const ListState st = ld_state(w.state + s);
            u32* hist = w.fb_hist + static_cast<u64>(s) * 3 * B;
            const ListState x = next_interval<THREADS>(st, B, ld_dev(&w.fb_above[s]), static_cast<u32>(a.slots[s].n), sh.wave, sh.pick, [&](u32 i) { return ld_dev(&hist[i]); });
            for (u32 i = tid; i < 3 * B; i += THREADS) st_dev(&hist[i], 0u);
            if (tid != 0) continue;
            st_state(w.state + s, x.a, x.b, x.rank, x.n, 0);
            if (x.a == x.b) {
                __hip_atomic_fetch_and(&w.open_of[g], ~(1u << j), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (x.rank < x.n) { or_dev(w.tie_of + g, 1u << j); add_dev(&w.fb->ties, 1u); }
            } else {
                add_dev(&w.fb->open[level + 1], 1u);
            }
        }
        meet(m);
    }

    bool counted = false;
    if constexpr (LONG) {                                  // ---- ties per chunk, where they lie gathered (one ranking)
        ListState st;
        counted = search && list_state(w, 0, &st) && list_ties_counted(a, st);         // uniform over all workgroups
        if (counted) {
            for (u64 c = c0 + tid; c < c1; c += THREADS) st_dev(&a.tiecnt[c], 0u);
            meet(m);
            for (u32 i = m.rank * THREADS + tid; i < st.n; i += m.size * THREADS) add_dev(&a.tiecnt[ld_dev(w.gidx + i) / kChunk], 1u);
            meet(m);
        }
    }
    if (!counted && (search || ld_dev(&w.fb->ties) != 0)) {              // ---- ties per chunk
        u32 cur = 0xFFFFFFFFu, mask = 0;
        for_chunks<LC, VEC, THREADS>(a, c0, c1, wanted(w.tie_of), [&](u64 c, const auto& ck) {
            const u32 g = group_of(c);
            if (g != cur) {                                // uniform
                cur = g;
                mask = ld_dev(&w.tie_of[g]);
                if (tid < static_cast<u32>(a.J)) {
                    ListState st{};
                    sh.a[tid] = ((mask >> tid) & 1u) && list_state(w, g * a.J + tid, &st) ? st.a : 0xFFFFFFFEu;
                }
            }
            if (tid < static_cast<u32>(a.J)) sh.count[tid] = 0;
            __syncthreads();
            for (u32 js = mask; js != 0; js &= js - 1u) {
                const u32 j = static_cast<u32>(__ffs(js)) - 1u, T = sh.a[j];
                if (T > 0x7FFFFFFFu) continue;             // uniform: no ties after all
                const u32 n = ck.equal(T);
                if (lane == 0 && n) atomicAdd(&sh.count[j], n);
            }
            __syncthreads();
            if (tid < static_cast<u32>(a.J)) st_dev(&a.tiecnt[static_cast<u64>(tid) * a.n_chunks + c], sh.count[tid]);
            __syncthreads();
            return false;
        });
        meet(m);
    }

    for (u32 f = m.rank; f < n_special; f += m.size) {     // ---- the tie rule, states and records
        const u32 s = ld_dev(w.special + f), g = s / a.J, j = s - g * a.J;
        ListState st;
        if (!list_state(w, s, &st)) continue;              // uniform
        const u32 T = st.a;
        Slot& slot = a.slots[s];
        u64 tie_end = slot.n;
        u32 last = 0xFFFFFFFFu;
        if (st.rank < st.n) {                              // uniform
            const u64 cb = a.per_tensor ? a.td[g].chunk_start : 0, ce = a.per_tensor ? a.td[g + 1].chunk_start : a.n_chunks;
            const u32* cnt = a.tiecnt + static_cast<u64>(j) * a.n_chunks;
            u32 cum = 0;
            if (tid == 0) { sh.pick[0] = static_cast<u32>(cb); sh.pick[1] = 0; sh.pick[2] = 0; }           // (found below; never out of range)
            __syncthreads();
            if constexpr (LONG) {
                constexpr u32 kAtOnce = 8;                 // chunks of a thread
                for (u64 b = cb; b < ce && cum < st.rank; b += kAtOnce * THREADS) {    // uniform
                    u32 x[kAtOnce], sum = 0, total;
#pragma unroll
                    for (u32 i = 0; i < kAtOnce; ++i) { const u64 c = b + kAtOnce * tid + i; x[i] = ld_dev(&cnt[c < ce ? c : ce - 1]); }
#pragma unroll
                    for (u32 i = 0; i < kAtOnce; ++i) { if (b + kAtOnce * tid + i >= ce) x[i] = 0; sum += x[i]; }
                    u32 before = cum + wg_incl_scan_u32<THREADS>(sum, sh.wave, &total) - sum;
#pragma unroll
                    for (u32 i = 0; i < kAtOnce; ++i) {
                        if (before < st.rank && st.rank <= before + x[i]) { sh.pick[0] = static_cast<u32>(b + kAtOnce * tid + i); sh.pick[1] = st.rank - before; }
                        before += x[i];
                    }
                    cum += total;
                }
            } else {
                for (u64 b = cb; b < ce && cum < st.rank; b += THREADS) {              // uniform
                    const u64 c = b + tid;
                    const u32 x = c < ce ? ld_dev(&cnt[c]) : 0u;
                    u32 total;
                    const u32 upto = cum + wg_incl_scan_u32<THREADS>(x, sh.wave, &total);
                    if (upto - x < st.rank && st.rank <= upto) { sh.pick[0] = static_cast<u32>(c); sh.pick[1] = st.rank - (upto - x); }
                    cum += total;
                }
            }
            __syncthreads();
            const u64 c = sh.pick[0];
            const u32 want = sh.pick[1];
            const TensorDesc& td = a.td[a.chunk_map[c]];
            constexpr int kRun = kChunk / THREADS;         // consecutive elements per thread
            const u64 e0 = (c - td.chunk_start) * kChunk + static_cast<u64>(tid) * kRun;
            u32 eq = 0;
#pragma unroll
            for (int x = 0; x < kRun; ++x)
                if (e0 + x < td.n && mag_key(LC ? lc_shift(td.w[e0 + x], td.lam[e0 + x], a.mu) : td.w[e0 + x]) == T) eq |= 1u << x;
            u32 total;
            const u32 mine = static_cast<u32>(__popc(eq)), before = wg_incl_scan_u32<THREADS>(mine, sh.wave, &total) - mine;
            if (before < want && want <= before + mine) {
                for (u32 skip = want - before - 1; skip > 0; --skip) eq &= eq - 1;
                sh.pick[2] = tid * kRun + static_cast<u32>(__ffs(eq)) - 1u;
            }
            __syncthreads();
            last = static_cast<u32>(c) * kChunk + sh.pick[2];
            tie_end = (c - td.chunk_start) * kChunk + sh.pick[2] + (a.per_tensor ? 0 : td.flat_start) + 1;
            __syncthreads();
        }
        if (tid == 0) {
            slot.remaining = st.rank; slot.n_tie = st.n; slot.need_tie = 0; slot.state = kDone;
            st_dev64(&slot.prefix, T);                     // the next phase reads these
            st_dev64(&slot.tie_end, tie_end);
            st_dev(&w.state[s].last, last);
            results[static_cast<u64>(j) * n_groups + g] = select_record(slot, true, T, st.rank, st.n, tie_end, (st.flags & kStateTied) ? slot.path : 3);
        }
    }
    if (!w.write) return;
    meet(m);

    const bool nnz = PQ && w.nnz_out != nullptr;
    if (n_apply != 0) {                                    // ---- the outputs
        u32 cur = 0xFFFFFFFFu, mask = 0, codes = 0;
        for_chunks<LC, VEC, THREADS>(a, c0, c1, wanted(w.apply_of), [&](u64 c, const auto& ck) {
            const u32 g = group_of(c);
            if (g != cur) {                                // uniform
                mask = ld_dev(&w.apply_of[g]);
                __syncthreads();
                if (tid < static_cast<u32>(a.J)) {
                    const Slot& slot = a.slots[static_cast<u64>(g) * a.J + tid];
                    sh.a[tid] = static_cast<u32>(ld_dev64(&slot.prefix));
                    sh.end[tid] = ld_dev64(&slot.tie_end);
                }
                __syncthreads();
                cur = g;
            }
            ck.template apply<PQ>(a, w.out, c, mask, sh.a, sh.end, vec_out != 0, &codes);
            return false;
        });
        if (nnz) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) codes += __shfl_xor(codes, d, 64);
            if (lane == 0 && codes != 0)
                __hip_atomic_fetch_add(&a.nnz_seg[(m.rank * (THREADS / 64) + (tid >> 6)) % kNnzSegs], static_cast<u64>(codes), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (tied) {                                            // ---- or the ties alone
        int nz = 0;
        const u32 per = n_special < m.size ? m.size / n_special : 1u, sub = m.rank % per;              // workgroups for each of them
        for (u32 f = m.rank / per; f < n_special && m.rank / per < m.size / per; f += m.size / per) {
            const u32 s = ld_dev(w.special + f), g = s / a.J, j = s - g * a.J;
            ListState st;
            if (!list_state(w, s, &st) || !(st.flags & kStateTied)) continue;          // uniform
            const u32 last = ld_dev(&w.state[s].last);
            const bool kept = st.a >= w.win[s].mid;        // what the sweep wrote for the ties
            const u32* gidx = w.gidx + static_cast<u64>(s) * w.gather_cap;
            constexpr int kB = 4;
            for (u32 i0 = sub * THREADS + tid; i0 < st.n; i0 += per * THREADS * kB) {
                u32 idx[kB];
                bool keep[kB], on[kB];
#pragma unroll
                for (int b = 0; b < kB; ++b) {
                    const u32 i = i0 + b * per * THREADS;
                    idx[b] = i < st.n ? ld_dev(gidx + i) : 0u;
                    keep[b] = idx[b] <= last;
                    on[b] = i < st.n && keep[b] != kept;
                }
                list_fix<LC, PQ, kB>(a, w, j, idx, keep, on, &nz);
            }
        }
        if (nnz && n_apply == 0) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) nz += __shfl_xor(nz, d, 64);
            if (lane == 0 && nz != 0)
                __hip_atomic_fetch_add(w.nnz_out, static_cast<u64>(static_cast<long long>(nz)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (nnz && n_apply != 0) {                             // ---- the count of non-zero codes
        meet(m);
        if (m.rank != 0) return;
        u32 v = 0, total;                                  // fewer than 2^32 together
        for (u32 i = tid; i < static_cast<u32>(kNnzSegs); i += THREADS) v += static_cast<u32>(ld_dev64(&a.nnz_seg[i]));
        wg_incl_scan_u32<THREADS>(v, sh.wave, &total);
        if (tid == 0) *w.nnz_out = total;
    }
}

constexpr int kSettleGrid = 512, kSettleThreads = 512;

// Several rankings, after k_list_gather.
template <bool VEC>
__global__ __launch_bounds__(kSettleThreads, 4) void k_list_settle(DataArgs a, ListArgs w, condensa_select* results, int n_groups, int vec_out) {
    __shared__ union { ListShared rank; u32 words[kFallbackWords]; } s_mem;           // one after the other
    ListShared& sh = s_mem.rank;
    u32* s_words = s_mem.words;
    __shared__ FallbackShared fs;
    __shared__ u32 s_tied, s_search;
    const u32 n_special = w.fb->special;                   // final: an earlier kernel counted
    const u32 n_r = static_cast<u32>(w.n_rankings), shares = n_r * 16 <= gridDim.x ? 16u : (n_r <= gridDim.x ? gridDim.x / n_r : 1u);
    for (u32 v = blockIdx.x; v < n_r * shares; v += gridDim.x) {
        const u32 s = v / shares;
        const u32 want = n_special != 0 && list_tied(w, s) ? 0u : w.bin_want[s];
        list_rank<false, false, kSettleThreads, false>(a, w, sh, s, want, w.gathered[static_cast<u64>(s) * kListLine], false, 0, v % shares, shares, results, n_groups);
    }
    if (n_special == 0) return;
    if (threadIdx.x == 0) { s_tied = 0; s_search = 0; }
    __syncthreads();
    for (u32 f = threadIdx.x; f < n_special; f += kSettleThreads) {
        const u32 s = w.special[f];
        if (!list_tied(w, s)) continue;
        s_tied = 1;
        if (w.state[s].rank < w.gathered[static_cast<u64>(s) * kListLine]) s_search = 1;
    }
    __syncthreads();
    const bool tied = s_tied != 0, search = s_search != 0;
    if (!tied && w.fb->apply == 0) return;                 // the same in every workgroup
    Meet m;
    if (!meet_join(m, w.meet, fs.pick)) return;
    list_fallback<false, VEC, false, false, kSettleThreads>(a, w, m, fs, s_words, results, n_groups, vec_out, tied, search);
}

// One ranking: everything after the sweep in one launch (k_list_hist, k_list_gather and k_list_settle took 22 us for the L-C step of
// 20 M weights, 18 for 2^20 weights pruned; this 14 and 11).  Every workgroup finds
// the threshold's bin for itself.  As a rule the bin's entries are few: the workgroups whose wavefronts have a segment of the
// list walk it, post the entries of the bin and settle those beside it, whichever posts last ranks them, and each settles its own; the
// others have left at once.  Otherwise (the list is incomplete, thousands of ties, a crowded window) all of them stay, register and
// go through the phases of list_fallback.
// Posting is one update that counts workgroups and entries both; the entries follow it, each with a bit that says it is there, and the
// last workgroup waits for those still on their way (their workgroups wait for nobody).
// Bound by latency: a launch and some ten dependent accesses.
// LONG: lists of millions of entries (list_long says which).  Four wavefronts share a segment, and bins of thousands are ranked in the same way.
template <bool LC, bool VEC, bool PQ, bool LONG>
__global__ __launch_bounds__(kSettleThreads, 4) void k_list_resolve(DataArgs a, ListArgs w, condensa_select* results, int vec_out) {
    constexpr u32 kWaves = kSettleThreads / 64, kRoom = 256, kFound = 64;              // for each wavefront
    static_assert(kMaxWalkers == kListSegs / kWaves && kMaxWalkers * kListParts <= static_cast<u32>(kSettleGrid), "a segment a wavefront");
    constexpr u32 kPosted = LONG ? kListPosted : kListFound, kParts = LONG ? kListParts : 1u;
    __shared__ union {                                     // one after the other
        ListShared rank;
        typename std::conditional<LONG, RankLong, RankShort>::type few;
        u32 words[kFallbackWords];
    } s_mem;
    __shared__ ListFindShared<kSettleThreads> find;
    __shared__ u32 s_queue[kWaves * kRoom], s_fkey[kWaves * kFound], s_fidx[kWaves * kFound];
    __shared__ FallbackShared fs;
    __shared__ u32 s_found[kWaves + 1];
    __shared__ u64 s_verdict[kWaves + 1];
    ListShared& sh = s_mem.rank;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const ListRank rk = w.rank[0];
    const ListWin win = w.win[0];
    const Slot& slot = a.slots[0];
    const u32 k = static_cast<u32>(slot.k), n_all = static_cast<u32>(slot.n);
    const ListFound f = list_find<kSettleThreads>(w, find, 0, rk, win, k);
    const bool nnz = PQ && w.nnz_out != nullptr && w.write;
    auto sweep_codes = [&]() {                             // the sweep's count of non-zero codes, in thread 0
        u32 v = 0, total;                                  // fewer than 2^32
        for (u32 i = tid; i < static_cast<u32>(kListSegs); i += kSettleThreads) v += w.nnz[i];
        wg_incl_scan_u32<kSettleThreads>(v, find.scratch, &total);
        return total;
    };
    auto add_corrections = [&](int nz, u64* to) {
        const u32 sum = wave_sum_u32(static_cast<u32>(nz));                            // modulo 2^32: the sum of a wavefront's is small
        if (lane == 0 && sum != 0)
            __hip_atomic_fetch_add(to, static_cast<u64>(static_cast<long long>(static_cast<int>(sum))), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // Nothing is kept, and the sweep kept nothing.  Not by slot.state: that is written in this launch, and a workgroup that starts
    // after the others are done would find it changed.
    if (k == 0) {                                          // uniform
        if (blockIdx.x != 0) return;
        if (nnz) { const u32 codes = sweep_codes(); if (tid == 0) *w.nnz_out = codes; }
        if (tid == 0) *results = select_record(slot, false, 0, 0, 0, 0, slot.path);
        return;
    }
    const bool crowded = win_crowded(win);
    int nz = 0;
    WaveQueue<kRoom> queue{s_queue + wave * kRoom, 0, win_mid_bin(win) > f.bin, win.lo, win_shift(win), f.bin, win_mid_bin(win)};
    if (!crowded && f.want != 0 && f.n_in <= kPosted) {               // the same in every workgroup
        const u32 part = blockIdx.x % kParts;              // (2.7 M entries, 1.2 G weights pruned: a wavefront a segment 30 us walked and 14 corrected, now 5 and 10)
        const u32 walkers = (rk.n_segs + kWaves - 1) / kWaves * kParts;  // at most the grid
        if (blockIdx.x >= walkers) return;
        u32* const fkey = s_fkey + wave * kFound;
        u32* const fidx = s_fidx + wave * kFound;
        auto post = [&](u32 at, u32 key, u32 idx) {
            if (at < kPosted) st_dev64(w.picked + at, kPicked | (static_cast<u64>(key) << 32) | idx);
        };
        u32 n_found = 0;                                   // uniform
        list_walk_own(w, rk, find.cnt, blockIdx.x / kParts * kWaves + wave, gridDim.x * kWaves, [&](bool there, u32 key, u32 idx) {
            const bool found = queue.template offer<LC, PQ>(a, w, 0, there, key, idx, &nz);
            const u64 m = __ballot(found);
            if (m == 0) return;                            // uniform
            const u32 count = static_cast<u32>(__popcll(m));
            if (n_found + count <= kFound) {
                if (found) { fkey[n_found + lanes_below(m)] = key; fidx[n_found + lanes_below(m)] = idx; }
                n_found += count;
                return;
            }
            u32 base = 0;                                  // no room
            if (lane == 0) base = add_dev(w.arrived, count) & 0xFFFFFu;
            base = __shfl(base, 0, 64);                    // by all lanes: one that lane 0 does not take part in returns 0
            if (found) post(base + lanes_below(m), key, idx);
        }, part, kParts);
        if (lane == 0) s_found[wave] = n_found;
        __syncthreads();
        u32 before = 0, all = 0;
#pragma unroll
        for (u32 i = 0; i < kWaves; ++i) { before += i < wave ? s_found[i] : 0u; all += s_found[i]; }
        if (tid == 0) s_found[kWaves] = add_dev(w.arrived, (1u << 20) | all);
        __syncthreads();
        const u32 ticket = s_found[kWaves], base = (ticket & 0xFFFFFu) + before;
        if (lane < n_found) post(base + lane, fkey[lane], fidx[lane]);
        if (tid == 0) st_dev(w.range + blockIdx.x, kRangeKnown | (all << kRangeBits) | ((ticket & 0xFFFFFu) < kPosted ? ticket & 0xFFFFFu : kPosted));
        if constexpr (!LONG) queue.template fix<LC, PQ>(a, w, 0, &nz);
        // what settling its own entries will read is on its way meanwhile
        const u32 idx1[1] = {lane < n_found ? fidx[lane] : 0u};
        bool on1[1] = {lane < n_found};
        FixLoads<LC, 1> loads;
        if (w.write && n_found != 0) list_fix_load<LC, 1>(a, w, 0, idx1, on1, loads);
        if ((ticket >> 20) + 1 == walkers) {               // uniform: the last one
            const u32 n_in = (ticket & 0xFFFFFu) + all;
            if constexpr (LONG) list_rank_long<LC, PQ, kSettleThreads>(a, w, rk, find.cnt, s_mem.few, f.want, n_in, f.bin, win, walkers, results, &nz);
            else                list_rank_short<LC, PQ, kSettleThreads>(a, w, rk, find.cnt, s_mem.few, f.want, n_in, f.bin, win, walkers, results, &nz);
        }
        // Long lists have hundreds of corrections for a wavefront, 40 to 80 us where its estimate is poor: the workgroup that ranks does its own last, or the
        // others, done with theirs, hear nothing for so long that they leave (604 M weights in rows of very different sizes, L-C step 2 205 -> 2 033 us).
        if constexpr (LONG) queue.template fix<LC, PQ>(a, w, 0, &nz);
        if (w.write && n_found != 0) {                     // uniform over the wavefront
            // The verdict comes from a workgroup that is running once all have posted; if some of them are not even running yet (another
            // launch holds the chip), this one does not keep them from it for long.
            u64 v = 0;
            if (lane == 0) {
                for (int polls = 0; polls < ((w.force & kForceNoVerdict) ? 0 : (LONG ? 192 : 64)) && ((v = ld_dev64(w.verdict + blockIdx.x)) & kPicked) == 0; ++polls) __builtin_amdgcn_s_sleep(4);
                if (w.force & kForceAsk) v = 0;
            }
            v = (static_cast<u64>(__shfl(static_cast<u32>(v >> 32), 0, 64)) << 32) | __shfl(static_cast<u32>(v), 0, 64);
            s_verdict[wave] = v;
        } else if (lane == 0) {
            s_verdict[wave] = kPicked;                     // asks for nothing
        }
        __syncthreads();
        bool stay = true;
#pragma unroll
        for (u32 i = 0; i < kWaves; ++i) stay = stay && (s_verdict[i] & kPicked) != 0;
        if (!stay) {                                       // uniform: leave the entries to the workgroup that ranks, unless it has just spoken
            if (tid == 0) {
                u64 was = 0;
                __hip_atomic_compare_exchange_strong(w.verdict + blockIdx.x, &was, kWalkerLeft, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_verdict[kWaves] = was;
            }
            __syncthreads();
            stay = (s_verdict[kWaves] & kPicked) != 0;
            if (stay) s_verdict[wave] = s_verdict[kWaves];
        }
        if (stay && w.write && n_found != 0) {
            const u64 v = s_verdict[wave];
            const u32 key = lane < n_found ? fkey[lane] : 0u, T = static_cast<u32>(v >> 32) & 0x7FFFFFFFu;
            const bool keep1[1] = {key > T || (key == T && idx1[0] <= static_cast<u32>(v))};
            on1[0] = on1[0] && keep1[0] != (key >= win.mid);
            list_fix_store<LC, PQ, 1>(a, loads, keep1, on1, &nz);
        }
        if (!nnz) return;
        // one update a workgroup: with one a wavefront, up to 1024 took turns at the counter (44 M weights: 31.6 us
        // for this launch, now 22.1)
        const u32 corrections = wave_sum_u32(static_cast<u32>(nz));                    // modulo 2^32: the workgroup's sum is small
        if (lane == 0) s_found[wave] = corrections;
        __syncthreads();
        if (tid == 0) {
            u32 sum = 0;
#pragma unroll
            for (u32 i = 0; i < kWaves; ++i) sum += s_found[i];
            if (sum != 0)
                __hip_atomic_fetch_add(&a.ctl->nnz_delta, static_cast<u64>(static_cast<long long>(static_cast<int>(sum))), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_dev();                                    // it is there before this workgroup counts as done
            s_found[kWaves] = add_dev(w.ended, 1u);
        }
        __syncthreads();
        if (s_found[kWaves] + 1 != walkers) return;        // uniform: the last one adds up
        const u32 codes = sweep_codes();
        if (tid == 0) *w.nnz_out = codes + ld_dev64(&a.ctl->nnz_delta);
        return;
    }
    Meet m;
    if (!meet_join(m, w.meet, fs.pick)) return;
    const bool first = m.rank == 0;
    bool gather = false;
    if (crowded) {
        if (first) list_leave<kSettleThreads>(a, w, 0, win.lo, win.hi, k, 0, kStateUnsure);
    } else {
        gather = list_leave_open<kSettleThreads>(a, w, 0, win, f, n_all, k, first);
    }
    if (first && tid == 0) st_dev(w.bin_want, gather ? f.want : 0u);
    if (first && nnz && gather) { const u32 codes = sweep_codes(); if (tid == 0) st_dev64(w.nnz_out, codes); }
    if (gather) {
        u32 most = 0, mostc = 0;
        list_gather_many<LC, PQ, kRoom>(a, w, 0, 0, rk, find.cnt, m.rank * kWaves + wave, m.size * kWaves, queue, &most, &mostc, &nz);
        if (mostc) { max_dev(w.gmax, most); max_dev(w.gmaxc, mostc); }
        queue.template fix<LC, PQ>(a, w, 0, &nz);
        if (nnz) add_corrections(nz, &a.ctl->nnz_delta);
    }
    meet(m);
    if (gather && !list_tied(w, 0)) {                      // the same in every workgroup
        const u32 shares = m.size < 16 ? m.size : 16u;
        if (m.rank < shares) list_rank<LC, PQ, kSettleThreads, true>(a, w, sh, 0, f.want, f.n_in, false, 0, m.rank, shares, results, 1);
        return;
    }
    if (first && nnz && gather && tid == 0) __hip_atomic_fetch_add(w.nnz_out, ld_dev64(&a.ctl->nnz_delta), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool tied = gather;
    list_fallback<LC, VEC, PQ, LONG, kSettleThreads>(a, w, m, fs, s_mem.words, results, 1, vec_out, tied, tied && f.want < f.n_in);
}

// The kernels that PER_TENSOR calls launch one after the other, so that they lie together in the code object: with others between them (that of long lists,
// strips) VGG-19 per layer took 72.6 us instead of 72.1 with every instruction the same, now 72.0.
template __global__ void k_begin_sample<false, true, false>(BeginSampleArgs, ListArgs);
template __global__ void k_list_sweep<false, true, 4, false>(DataArgs, ListArgs);
template __global__ void k_list_settle<true>(DataArgs, ListArgs, condensa_select*, int, int);

}  // namespace condensa
