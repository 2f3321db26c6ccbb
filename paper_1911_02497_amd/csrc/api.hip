// C-ABI entry points of the compression-step library (see include/condensa.h): argument checks,
// table building, workspace carving and the kernel launch sequences.
#include <chrono>
#include <memory>
#include <thread>

#include "host.h"
#include "k_apply.h"
#include "k_quantize.h"
#include "k_fused.h"
#include "k_select.h"
#include "k_listed.h"
#include "k_structure.h"
#include "k_window.h"
#include "k_struct_fused.h"
#include "k_struct_list.h"
#include "k_struct_strip.h"

namespace condensa {

std::atomic<int> g_last_hip_error{0};
std::atomic<uint64_t> g_launches{0};
static thread_local u32 t_force = 0;

// ---- configuration ---------------------------------------------------------------------------------

namespace {
// process-wide defaults: what a NULL condensa_config stands for
std::atomic<int64_t> g_options[CONDENSA_OPT_COUNT] = {{0}, {0}, {80}, {0}, {0}, {0}, {0}};

bool option_value_ok(int option, int64_t value) {
    if (value < 0) return false;
    switch (option) {
        case CONDENSA_OPT_SELECT_PATH:   return value <= 2;
        case CONDENSA_OPT_SAMPLE_LOG2:   return value == 0 || (value >= 10 && value <= 26);
        case CONDENSA_OPT_WINDOW_MARGIN: return value <= 0x7FFFFFFF;
        case CONDENSA_OPT_CAND_SHIFT:    return value <= 30;
        case CONDENSA_OPT_PROFILE:       return value < (1 << CONDENSA_PHASE_COUNT);
        case CONDENSA_OPT_APPLY_THREADS: return value == 0 || value == 64 || value == 128 || value == 256;
        case CONDENSA_OPT_FUSED_SWEEP:   return value <= 1;
        default: return false;
    }
}
}  // namespace

condensa_status set_default_option(int option, int64_t value) {
    if (!option_value_ok(option, value)) return CONDENSA_ERR_ARG;
    g_options[option].store(value);
    return CONDENSA_OK;
}

condensa_status resolve_config(const condensa_config* c, Config* out) {
    if (c == nullptr) {
        for (int i = 0; i < CONDENSA_OPT_COUNT; ++i) out->v[i] = g_options[i].load();
        return CONDENSA_OK;
    }
    if (c->reserved != 0) return CONDENSA_ERR_ARG;
    const int64_t v[CONDENSA_OPT_COUNT] = {c->select_path, c->sample_log2, c->window_margin, c->cand_shift,
                                           c->profile, c->apply_threads, c->fused_sweep};
    for (int i = 0; i < CONDENSA_OPT_COUNT; ++i) {
        if (!option_value_ok(i, v[i])) return CONDENSA_ERR_ARG;
        out->v[i] = v[i];
    }
    return CONDENSA_OK;
}

// ---- pinned staging slots --------------------------------------------------------------------------

namespace {
// The slots' words and their first kStageBytes each are one pinned block, allocated on the first call; a larger image
// gets a buffer of its own, which stays with the slot.  A slot is free when it is not being filled and the device
// has stored the ticket of its last use.  A call that finds none waits (the host is 32 calls ahead), but not for ever: its
// tables then travel as kernel arguments, whose launches report an error of the device.
constexpr int kStageSlots = 32;
constexpr size_t kStageBytes = 64u << 10;
constexpr std::chrono::milliseconds kStageWait{100};
constexpr unsigned kStageFlags = hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent;
struct Stage {
    char* big = nullptr;
    size_t big_cap = 0;
    u64 ticket = 0;
    bool filling = false;
};
Stage g_stage[kStageSlots];
char* g_stage_block = nullptr;                // [kStageSlots] words of 64 bytes, then [kStageSlots] images
int g_stage_next = 0;
std::mutex g_stage_mu;

u64* stage_done(int i) { return reinterpret_cast<u64*>(g_stage_block + static_cast<size_t>(i) * 64); }
}  // namespace

condensa_status StageImage::acquire(size_t bytes, hipStream_t stream) {
    if (tried_) return CONDENSA_OK;
    tried_ = true;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess) (void)hipGetLastError();
    if (capture != hipStreamCaptureStatusNone) return CONDENSA_OK;
    std::unique_lock<std::mutex> lock(g_stage_mu);
    if (g_stage_block == nullptr) {
        void* p = nullptr;
        CONDENSA_HIP(hipHostMalloc(&p, kStageSlots * (64 + kStageBytes), kStageFlags));
        std::memset(p, 0, kStageSlots * 64);
        g_stage_block = static_cast<char*>(p);
    }
    int found = -1;
    const auto give_up = std::chrono::steady_clock::now() + kStageWait;
    for (int tries = 0;; ++tries) {
        for (int k = 0; k < kStageSlots; ++k) {
            const int i = (g_stage_next + k) % kStageSlots;
            if (g_stage[i].filling || __atomic_load_n(stage_done(i), __ATOMIC_ACQUIRE) != g_stage[i].ticket) continue;
            if (found < 0) found = i;
            if (bytes <= kStageBytes || g_stage[i].big_cap >= bytes) { found = i; break; }     // one that needs no new buffer
        }
        if (found >= 0) break;
        // every slot is in flight: the device is behind, or does not answer
        lock.unlock();
        if (tries < 2000) {
            std::this_thread::yield();
        } else {
            if (std::chrono::steady_clock::now() > give_up) return CONDENSA_OK;
            std::this_thread::sleep_for(std::chrono::microseconds(20));
        }
        lock.lock();
    }
    Stage& s = g_stage[found];
    if (bytes > kStageBytes && s.big_cap < bytes) {
        if (s.big) CONDENSA_HIP(hipHostFree(s.big));
        s.big = nullptr;
        s.big_cap = 0;
        void* p = nullptr;
        CONDENSA_HIP(hipHostMalloc(&p, align_up(bytes, 4096), kStageFlags));
        s.big = static_cast<char*>(p);
        s.big_cap = align_up(bytes, 4096);
    }
    if (bytes <= kStageBytes) g_stage_next = (found + 1) % kStageSlots;      // large images keep to the slots that have a buffer
    s.filling = true;
    slot_ = found;
    data_ = bytes > kStageBytes ? s.big : g_stage_block + kStageSlots * 64 + static_cast<size_t>(found) * kStageBytes;
    done_ = stage_done(found);
    ticket_ = s.ticket + 1;
    return CONDENSA_OK;
}

void StageImage::commit() {
    if (slot_ < 0) return;
    std::lock_guard<std::mutex> lock(g_stage_mu);
    g_stage[slot_].filling = false;
    g_stage[slot_].ticket = ticket_;
    slot_ = -1;
}

// Not committed.  Once a launch was attempted the kernel may be in the stream whatever was reported: the error can be one
// that the thread had left behind.  The slot is then free when the stream has been waited for, at whichever ticket the
// device left; if the stream itself has failed, it stays out of the pool.
StageImage::~StageImage() {
    if (slot_ < 0) return;
    const bool drained = !launched_ || hipStreamSynchronize(stream_) == hipSuccess;
    if (!drained) { (void)hipGetLastError(); return; }
    std::lock_guard<std::mutex> lock(g_stage_mu);
    g_stage[slot_].ticket = __atomic_load_n(stage_done(slot_), __ATOMIC_ACQUIRE);
    g_stage[slot_].filling = false;
}

// ---- phase timing ----------------------------------------------------------------------------------

namespace {
struct Interval {
    hipEvent_t a = nullptr, b = nullptr;
    int phase = 0;
};
std::vector<Interval> g_intervals;          // both events recorded, not yet read
std::vector<hipEvent_t> g_event_pool;
double g_phase_ms[CONDENSA_PHASE_COUNT] = {};
u64 g_phase_n[CONDENSA_PHASE_COUNT] = {};
std::mutex g_prof_mu;

hipEvent_t take_event() {                   // g_prof_mu held
    if (!g_event_pool.empty()) {
        hipEvent_t e = g_event_pool.back();
        g_event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}
}  // namespace

PhaseTimer::PhaseTimer(int phase, hipStream_t stream, const Config& cfg) : phase_(phase), stream_(stream) {
    if (((cfg[CONDENSA_OPT_PROFILE] >> phase) & 1) == 0) return;
    hipEvent_t a, b;
    {
        std::lock_guard<std::mutex> lock(g_prof_mu);
        a = take_event();
        b = take_event();
    }
    if (a && b && hipEventRecord(a, stream_) == hipSuccess) {
        a_ = a;
        b_ = b;
        return;
    }
    std::lock_guard<std::mutex> lock(g_prof_mu);
    if (a) g_event_pool.push_back(a);
    if (b) g_event_pool.push_back(b);
}

PhaseTimer::~PhaseTimer() {
    if (!a_) return;
    const bool ok = hipEventRecord(b_, stream_) == hipSuccess;
    std::lock_guard<std::mutex> lock(g_prof_mu);
    if (ok) {
        Interval iv;
        iv.a = a_; iv.b = b_; iv.phase = phase_;
        g_intervals.push_back(iv);
    } else {
        g_event_pool.push_back(a_);
        g_event_pool.push_back(b_);
    }
}

// ---- workspace layout ----------------------------------------------------------------------------

static u64 window_sample_size(u64 N, const Config& cfg) {
    const int64_t opt = cfg[CONDENSA_OPT_SAMPLE_LOG2];
    u64 s;
    if (opt > 0) s = static_cast<u64>(1) << (opt > 26 ? 26 : opt);
    else {
        s = N / 8;
        if (s < (1u << 18)) s = 1u << 18;
        if (s > (1u << 21)) s = 1u << 21;
    }
    s = (s + kSampleUnit - 1) / kSampleUnit * kSampleUnit;
    return s;
}

static u64 window_cand_capacity(u64 N, int J, const Config& cfg) {
    const int64_t opt = cfg[CONDENSA_OPT_CAND_SHIFT];
    const int shift = (opt > 0 && opt < 40) ? static_cast<int>(opt) : (J > 1 ? 3 : 5);
    u64 c = N >> shift;
    if (c < 4096) c = 4096;
    return c;
}

// Which selection a call takes when its configuration does not say.  Listed windows (k_listed.h): PER_TENSOR scope and
// several densities while the lists' 32-bit indices last (four densities: 2^26 weights 209 us against 461 with the
// windows of several densities and 417-500 with radix levels, 2^28 weights 726 against 1152 and 1954).  One density: up to
// 2^31 weights (density 0.1, listed and sampled: pruning 2^27 weights 232 and 316 us, 2^28 418 and 507, 2^29 840 and 899, 1.2 G 1746 and 1878; L-C step
// 481 and 567, 941 and 997, 1917 and 2006, 3797 and 3921).  Sampled window (k_window.h, k_fused.h): one density beyond that line, where the list would
// hold more than its workgroups settle quickly, several beyond 32-bit indices.  Radix levels: where neither applies.
static bool list_fits(u64 N, int n_tensors, int n_slots) {
    return N > 0 && n_slots <= kListMaxRankings && N + static_cast<u64>(n_tensors) * kChunk < (static_cast<u64>(1) << 32);
}
static bool want_list(u64 N, int n_tensors, int n_slots, bool per_tensor, int J, const Config& cfg) {
    if (cfg[CONDENSA_OPT_SELECT_PATH] != 0 || !list_fits(N, n_tensors, n_slots)) return false;
    return per_tensor || J > 1 || N < (static_cast<u64>(1) << 31);
}
static bool want_window(u64 N, int n_tensors, bool per_tensor, int J, const Config& cfg) {
    if (per_tensor) return false;
    if ((N >> kCandTensorShift) != 0) return false;        // candidates carry their tensor above a 44-bit flat index
    const int64_t mode = cfg[CONDENSA_OPT_SELECT_PATH];
    if (mode == 1) return false;
    if (mode == 2) return N >= 1;
    return N > 0 && !want_list(N, n_tensors, J, per_tensor, J, cfg);
}

// One density whose selection is a sweep of its own (an output in place of an input, two sweeps asked for, no outputs): the listed windows' sweep then
// writes nothing but its list, and the sampled window's own sweep does that faster where there are many weights, its launches being paid for.  L-C steps in
// place, density 0.1, listed and sampled: 2.4 10^8 weights 1193 and 1159 us, 3.2 10^8 1524 and 1454, 1.2 G 5810 and 5341; from 3 2^26 on (where lists
// of one sweep begin to be worth more than windows).  Pruning in place and selection alone: 3.2 10^8 weights 727 and 755, 305 and 332; 8 10^8 1770 and 1739,
// 682 and 670 (density 0.6: 1800 and 1836, 698 and 744); 1.66 G 3790 and 3639, 1442 and 1315; from 2^29 on.  A workspace without room for it: listed windows.
static void prefer_window_for_two_sweeps(int op, u64 N, int n_tensors, size_t workspace_bytes, Config* cfg, Layout* L) {
    const u64 from = op == CONDENSA_OP_LC_STEP ? static_cast<u64>(3) << 26 : static_cast<u64>(1) << 29;
    if (!L->listed || (*cfg)[CONDENSA_OPT_SELECT_PATH] != 0 || N < from) return;
    Config sampled = *cfg;
    sampled.v[CONDENSA_OPT_SELECT_PATH] = 2;
    const Layout W = make_layout(op, N, 0, n_tensors, 1, CONDENSA_SCOPE_GLOBAL, sampled);
    if (workspace_bytes < W.total) return;
    *cfg = sampled;
    *L = W;
}

// A workspace may have room for the lists with fewer gathered entries alone (sized for several densities, which an L-C step does not have, or by hand).
static void fewer_gathered_where_short(int op, u64 N, int n_tensors, int J, int scope, size_t workspace_bytes, const Config& cfg, Layout* L) {
    if (L->l_gather_cap > kListGather && workspace_bytes < L->total) *L = make_layout(op, N, 0, n_tensors, J, scope, cfg, false, true);
}

// Segments of the rankings' lists: what their sweep's wavefronts call for (elements per wavefront).
static u64 list_wave_elems(u64 N, int J, bool lc) { return 256u * static_cast<u64>(J > 1 ? list_multi_quads(N) : (lc ? kFusedQuadsLC : kFusedQuadsPrune)); }
static u32 list_max_segs(u64 n, int n_slots, int J, bool lc) {
    u32 most = J > 1 ? 256u : static_cast<u32>(kListSegs);
    while (most > 16 && static_cast<u64>(most) * n_slots > (1u << 16)) most /= 2;        // many rankings share the atomics' rate
    return list_segments(n, list_wave_elems(n, J, lc), most);
}
// List entries of one ranking, a multiple of kListRow n_segs; and the most that the rankings of one density can add up
// to when the tensors' sizes are not known yet.
static u64 list_entries(u64 n, u32 n_segs, const Config& cfg) {
    const u64 unit = static_cast<u64>(kListRow) * n_segs;
    return (list_capacity(n, static_cast<int>(cfg[CONDENSA_OPT_CAND_SHIFT])) + unit - 1) / unit * unit;
}
static u64 list_entries_bound(u64 N, int n_tensors, bool per_tensor, u32 max_segs, const Config& cfg) {
    if (!per_tensor) return list_entries(N, max_segs, cfg);
    const u64 nt = static_cast<u64>(n_tensors);
    const int64_t shift = cfg[CONDENSA_OPT_CAND_SHIFT];
    u64 most = shift > 0 ? (N >> shift) + 4096 * nt : N / 4 + 4096 * nt;          // list_capacity is at most n / 4 + 4096,
    if (shift <= 0 && N / 48 + (nt << 18) < most) most = N / 48 + (nt << 18);     // at most n / 48 + 2^18,
    if (shift <= 0 && N < most) most = N;                                         // and at most n
    return most + static_cast<u64>(kListRow) * max_segs * nt;
}
// Bins of list_fallback's histograms: all of one population's in 48 KB of LDS, all rankings' in 12 MB, and no more than a
// workgroup searches quickly (an interval ends at the keys that are there, so ties take one level whatever the number).
static u32 list_fallback_bins(int n_slots, int J) {
    u32 bins = 1024;
    while (3 * bins * static_cast<u32>(J) > kFallbackWords) bins /= 2;
    while (bins > 256 && static_cast<u64>(bins) * static_cast<u64>(n_slots) > (1u << 20)) bins /= 2;
    return bins;
}
// Copies of a ranking's histogram (list_hist_copy): what the sweep's updates ask for, and 256 KB for all rankings.
static u32 list_hist_copies(int n_slots) {
    u32 c = 16;
    while (c > 1 && c * static_cast<u32>(n_slots) > 256) c /= 2;
    return c;
}
// One ranking: posted entries, verdicts and ranges (ListArgs::picked and what follows it).  Those of long lists lie where gathered entries otherwise
// do (posted they are not gathered), cleared that far, so that such calls ask for no more workspace than when their bins were short.
static u32 list_posted(u64 N) { return list_long(N) ? kListPosted : kListFound; }
static u32 list_walkers(u64 N) { return list_long(N) ? kMaxWalkers * kListParts : kMaxWalkers; }
static size_t list_post_bytes(u64 N) { return (list_posted(N) + list_walkers(N)) * sizeof(u64) + list_walkers(N) * sizeof(u32); }
static_assert((kListPosted + kMaxWalkers * kListParts) * sizeof(u64) + kMaxWalkers * kListParts * sizeof(u32) <= kListGather * sizeof(u32), "gathered keys make room");
static u32 list_uneven_copies(int n_slots) { return n_slots == 1 ? 64u : list_hist_copies(n_slots); }
static u32 list_groups(u64 n, int J, bool per_tensor, const Config& cfg) {         // sampling workgroups of a population
    const int64_t opt = cfg[CONDENSA_OPT_SAMPLE_LOG2];
    if (opt <= 0) return list_sample_groups(n, J, per_tensor);
    if ((static_cast<u64>(1) << opt) <= static_cast<u64>(kListThreads) * kListUnits * kSampleUnit) return 1;
    u32 w = 32;                                            // fewer draws would not tell their deviation
    while (w < static_cast<u32>(kListMaxW) && static_cast<u64>(w) * kListThreads * kSampleUnit < (static_cast<u64>(1) << opt)) w *= 2;
    return w;
}

// Block pruning in strips: sampling workgroups, blocks that each draws, and bins over the window: a few blocks to each of a bin's places.
constexpr u64 kStripMostBlocks = static_cast<u64>(1) << 24, kStripMostElems = static_cast<u64>(1) << 30;
struct StripBins { u32 log_bins, log_room; };
static u32 strip_groups(u64 F) { return F < (1u << 17) ? 32u : (F < (1u << 18) ? 64u : (F < (1u << 20) ? 128u : 256u)); }
// Rounds of draws: a second one, some 8 us, where there are so many blocks that a narrower window is worth it, and where the threshold is among the first
// or last three of 128 draws, which would leave it unbounded (the fallback takes 15-20 us).
static u32 strip_rounds(u64 F, u64 k) { return F >= (1u << 22) || (k < F - k ? k : F - k) < F / 50 ? 2u : 1u; }
static StripBins strip_bins(u64 F) {
    const double draws = static_cast<double>(strip_groups(F)) * strip_rounds(F, F / 2) * kStripSample;
    const double listed = 8.0 * static_cast<double>(F) / std::sqrt(draws);             // in the window of a threshold in the middle, at the most
    StripBins b{8, 5};
    while ((1u << b.log_bins) < kStripMostBins && listed / 24 > static_cast<double>(1u << b.log_bins)) ++b.log_bins;
    while ((kStripCopies << b.log_room) < kStripMostSlots && listed > 0.75 * static_cast<double>(1u << (b.log_bins + b.log_room))) ++b.log_room;
    return b;
}

Layout make_layout(int op, u64 N, u64 F, int n_tensors, int J, int scope, const Config& cfg, bool no_window, bool few_gathered) {
    Layout L;
    const bool per_tensor = (scope == CONDENSA_SCOPE_PER_TENSOR);
    const bool structure = (op == CONDENSA_OP_FILTER_PRUNE || op == CONDENSA_OP_BLOCK_PRUNE);
    if (structure || op == CONDENSA_OP_LC_STEP) J = 1;
    L.n_groups = per_tensor ? (n_tensors > 0 ? n_tensors : 1) : 1;
    L.n_slots = L.n_groups * J;
    L.max_chunks = N / kChunk + static_cast<u64>(n_tensors);
    L.max_schunks = F / kChunk + static_cast<u64>(n_tensors);
    size_t off = 0;
    L.td = off;     off += align_up(static_cast<size_t>(n_tensors + 1) * sizeof(TensorDesc));
    L.out = off;    off += align_up(static_cast<size_t>(J) * (n_tensors > 0 ? n_tensors : 1) * sizeof(OutDesc));
    L.slots = off;  off += align_up(static_cast<size_t>(L.n_slots) * sizeof(Slot) + (structure ? 3 : 2 * kMaxJ) * sizeof(Slot));
    L.upload_bytes = off;
    const bool element = op == CONDENSA_OP_PRUNE || op == CONDENSA_OP_LC_STEP;
    if (element && !no_window && want_list(N, n_tensors, L.n_slots, per_tensor, J, cfg)) {
        const u64 nt = static_cast<u64>(n_tensors);
        const u64 groups = per_tensor ? (cfg[CONDENSA_OPT_SAMPLE_LOG2] > 0 ? nt * kListMaxW : nt + (N >> (J > 1 ? 11 : 13)) + kListMaxW) : list_groups(N, J, per_tensor, cfg);
        L.l_max_segs = list_max_segs(N, L.n_slots, J, op == CONDENSA_OP_LC_STEP);
        const u64 entries = static_cast<u64>(J) * list_entries_bound(N, n_tensors, per_tensor, L.l_max_segs, cfg);
        L.listed = true;
        L.l_rank = off;    off += align_up(static_cast<size_t>(L.n_slots) * sizeof(ListRank) + (per_tensor ? groups * sizeof(u32) : 0));
        L.zero_begin = off;
        L.ctl = off;       off += align_up(sizeof(Control));
        L.l_cnt = off;     off += align_up(static_cast<size_t>(L.n_slots) * L.l_max_segs * sizeof(u64));
        L.l_nnz = off;     off += align_up(kListSegs * sizeof(u32));
        L.seg = off;       off += op == CONDENSA_OP_LC_STEP ? align_up(kNnzSegs * sizeof(u64)) : 0;
        L.l_hist = off;    off += align_up(static_cast<size_t>(L.n_slots) * list_uneven_copies(L.n_slots) * kListBins * sizeof(u32));
        const bool long_list = L.n_slots == 1 && list_long(N);
        L.l_post = off;    off += L.n_slots == 1 ? align_up(256 + (long_list ? 0 : list_post_bytes(N))) : 0;
        L.l_gathered = off; off += align_up(static_cast<size_t>(L.n_slots) * kListLine * sizeof(u32));
        L.l_fb = off;      off += align_up(sizeof(FallbackCtl));
        L.l_gmax = off;    off += align_up(2 * static_cast<size_t>(L.n_slots) * sizeof(u32));
        L.l_masks = off;   off += align_up(3 * static_cast<size_t>(L.n_groups) * sizeof(u32));
        L.l_meet = off;    off += align_up(kMeetWords * sizeof(u32));
        const u32 gather = long_list && !per_tensor && !few_gathered ? kListGatherLong : kListGather;
        L.l_gather_cap = (1u << 20) / L.n_slots > gather ? gather : ((1u << 20) / L.n_slots < kListRanked ? kListRanked : (1u << 20) / L.n_slots);
        L.l_gkey = off;
        L.l_posted = long_list ? L.l_gkey : L.l_post + 256;
        L.zero_bytes = off - L.zero_begin + (long_list ? align_up(list_post_bytes(N)) : 0);
        off += align_up(static_cast<size_t>(L.n_slots) * L.l_gather_cap * sizeof(u32));
        L.chunk_map = off; off += align_up(static_cast<size_t>(L.max_chunks + 1) * sizeof(u32));
        L.tiecnt = off;    off += align_up(static_cast<size_t>(J) * L.max_chunks * sizeof(u32));
        L.l_special = off; off += align_up(2 * static_cast<size_t>(L.n_slots) * sizeof(u32));
        L.l_state = off;   off += align_up(static_cast<size_t>(L.n_slots) * sizeof(ListState));
        L.l_fb_bins = list_fallback_bins(L.n_slots, J);
        L.l_fb_hist = off; off += align_up(3 * static_cast<size_t>(L.n_slots) * L.l_fb_bins * sizeof(u32));
        L.l_want = off;    off += align_up(static_cast<size_t>(L.n_slots) * sizeof(u32));
        L.l_gidx = off;    off += align_up(static_cast<size_t>(L.n_slots) * L.l_gather_cap * sizeof(u32));
        L.l_win = off;     off += align_up(static_cast<size_t>(L.n_slots) * sizeof(ListWin));
        L.l_sorted = off;  off += J > 1 ? align_up(static_cast<size_t>(L.n_groups) * sizeof(ListSorted)) : 0;
        L.l_local = off;   off += align_up(static_cast<size_t>(groups) * J * 3 * sizeof(u64));
        L.l_key = off;     off += align_up(static_cast<size_t>(entries) * sizeof(u32));
        L.l_idx = off;     off += align_up(static_cast<size_t>(entries) * sizeof(u32));
        L.cand_cap = entries;
        L.sample_cap = groups;
        L.total = off;
        return L;
    }
    L.zero_begin = off;
    L.ctl = off;    off += align_up(sizeof(Control));
    L.hist0 = off;  off += align_up(static_cast<size_t>(L.n_groups) * kBins * sizeof(u64));
    // later-level histograms of the rankings over the data (one per ranking and level under GLOBAL scope),
    // then the window path's: candidate rankings [3][J], the sample's boundary rankings [2][2J + 1] and its
    // shared level 0 (see make_window_args)
    size_t n_hx = 2u * static_cast<size_t>(L.n_slots);
    if (!structure && !per_tensor) n_hx += 3u * J + 2u * (2u * J + 1u) + 1u;
    // structures under GLOBAL scope: one histogram per level of the 63-bit ranking, then (one-sweep block pruning) the
    // block sample's boundary rankings [2][3] and their shared level 0
    if (structure && !per_tensor) n_hx = kStructLevels + 2u * 3u + 1u;
    L.histx = off;  off += align_up(n_hx * kBins * sizeof(u64));
    // coarse sums of every histogram from hist0 on (the two regions above are contiguous: their sizes are multiples of 16 KB)
    L.histc = off;  off += align_up((static_cast<size_t>(L.n_groups) + n_hx) * kCoarse * sizeof(u64));
    if (!structure && !per_tensor) { L.seg = off; off += align_up(static_cast<size_t>(kSegs) * (2 + kMaxJ) * sizeof(u64)); }
    if (structure && !per_tensor) { L.seg = off; off += align_up(static_cast<size_t>(kSegs) * 2 * sizeof(u64)); }
    // per-chunk tie counts and the flags of the chunks that can hold ties: cleared with the counters, because the
    // tie search only visits flagged chunks and leaves the others' counts alone
    const u64 tie_chunks = structure ? L.max_schunks : ((op == CONDENSA_OP_COUNT_NONZERO || op == CONDENSA_OP_LC_SGD_STEP) ? 0 : L.max_chunks);
    L.tiecnt = off; off += align_up(static_cast<size_t>(J) * tie_chunks * sizeof(u32));
    if (!structure) { L.tiehit = off; off += align_up(static_cast<size_t>(tie_chunks + 1) * sizeof(u32)); }
    const bool tie_lists = !structure && !per_tensor && tie_chunks > 0;
    if (tie_lists) { L.tl_cnt = off; off += align_up(static_cast<size_t>(kMaxJ) * sizeof(u64)); }
    L.zero_bytes = off - L.zero_begin;
    L.chunk_map = off; off += align_up(static_cast<size_t>(L.max_chunks + 1) * sizeof(u32));
    if (tie_lists) {
        const u64 entries = static_cast<u64>(J) * kTieListCap;
        L.tl_key = off; off += align_up(static_cast<size_t>(entries) * sizeof(u32));
        L.tl_idx = off; off += align_up(static_cast<size_t>(entries) * sizeof(u64));
    }
    if (structure) {
        L.skeys = off;  off += align_up(static_cast<size_t>(F) * sizeof(u64));
        L.sblock = off; off += align_up(static_cast<size_t>(F / kBlock + 2) * sizeof(u32));
        L.smask = off;  off += align_up(static_cast<size_t>(F) + 1);
        if (!per_tensor) {                                  // one-sweep block pruning: sample keys and the list of window blocks
            u64 sc = F / 8;
            sc = sc < (1u << 12) ? (1u << 12) : (sc > (1u << 17) ? (1u << 17) : sc);
            L.sample_cap = sc;
            // room for an eighth of the blocks, and for all of them while that costs under a megabyte
            L.cand_cap = F / 8;
            if (L.cand_cap < (1u << 16)) L.cand_cap = F < (1u << 16) ? (F < 4096 ? 4096 : F) : (1u << 16);
            if (F <= kSmallCallElems && L.cand_cap < F) L.cand_cap = F;   // the list of k_struct_list.h holds every structure
            L.sample = off;   off += align_up(L.sample_cap * sizeof(u32));
            L.cand_key = off; off += align_up(L.cand_cap * sizeof(u32));      // ids of the listed blocks
            L.cand_idx = off; off += align_up(L.cand_cap * sizeof(u64));      // their aggregate keys
            if (op == CONDENSA_OP_BLOCK_PRUNE && cfg[CONDENSA_OPT_SELECT_PATH] == 0 && F > kSmallGroup && F <= kStripMostBlocks && N <= kStripMostElems) {
                const StripBins sb = strip_bins(F);
                const size_t bins = static_cast<size_t>(1) << sb.log_bins, slots = bins * kStripCopies << sb.log_room;
                L.strips = true;
                L.s_zero = off;
                L.s_hist = off;   off += align_up(bins * kStripCopies * sizeof(u32));
                L.s_above = off;  off += align_up(kStripAboves * kListLine * sizeof(u32));
                L.s_meet = off;   off += align_up(kMeetWords * sizeof(u32));
                L.s_pass = off;   off += align_up(3 * kStripPassWords * sizeof(u32));
                L.s_coarse = off; off += align_up((F / 64 + 2) * kListLine * sizeof(u32));
                L.s_win = off;    off += align_up(sizeof(ListWin));
                L.s_local = off;  off += align_up(3 * static_cast<size_t>(strip_groups(F)) * sizeof(u64));
                L.s_key = off;    off += align_up(slots * sizeof(u64));
                L.s_id = off;     off += align_up(slots * sizeof(u32));
                L.s_share = off;  off += align_up(2 * kStripResolveGrid * sizeof(u32) + sizeof(u64));
            }
        }
    } else if (!per_tensor && !no_window && op != CONDENSA_OP_COUNT_NONZERO && op != CONDENSA_OP_LC_SGD_STEP) {
        L.sample_cap = window_sample_size(N, cfg);
        L.cand_cap = window_cand_capacity(N, J, cfg);
        L.sample = off;   off += align_up(L.sample_cap * sizeof(u32));
        L.cand_key = off; off += align_up(L.cand_cap * sizeof(u32));
        L.cand_idx = off; off += align_up(L.cand_cap * sizeof(u64));
        L.sorted_windows = off; off += align_up(256);             // SortedWindows (196 B)
        if (J == 1) {
            L.cand_w = off;   off += align_up(L.cand_cap * sizeof(float));
            L.cand_lam = off; off += align_up(L.cand_cap * sizeof(float));
        }
    }
    L.total = off;
    return L;
}

// ---- tables ---------------------------------------------------------------------------------------

// Host memory of one call's tables.  The usual entry points take it from the heap; the entry point for
// callers that cannot allocate hands out pieces of a fixed buffer on its own stack instead.
class HostArena {
public:
    HostArena() = default;                                         // heap
    HostArena(char* fixed, size_t bytes) : fixed_(fixed), left_(bytes) {}
    HostArena(const HostArena&) = delete;
    HostArena& operator=(const HostArena&) = delete;
    // n zero-initialised objects of T (trivially copyable table types), or nullptr when a fixed buffer is used up
    template <typename T>
    T* array(size_t n) {
        const size_t bytes = align_up((n ? n : 1) * sizeof(T), 64);
        char* p;
        if (fixed_) {
            if (bytes > left_) return nullptr;
            p = fixed_;
            fixed_ += bytes;
            left_ -= bytes;
        } else {
            heap_.emplace_back(new char[bytes]);
            p = heap_.back().get();
        }
        std::memset(p, 0, bytes);
        return reinterpret_cast<T*>(p);
    }
private:
    char* fixed_ = nullptr;
    size_t left_ = 0;
    std::vector<std::unique_ptr<char[]>> heap_;
};

struct Tables {
    TensorDesc* td = nullptr;        // n_tensors + 1 (sentinel)
    int n_td = 0;
    u64 N = 0, n_chunks = 0, F = 0, n_schunks = 0;
    bool vec = true;
};

static condensa_status build_tensor_table(const condensa_tensor* tensors, int n_tensors, Tables* tb, HostArena& arena) {
    if (n_tensors < 0 || n_tensors > CONDENSA_MAX_TENSORS) return CONDENSA_ERR_SIZE;
    if (n_tensors > 0 && tensors == nullptr) return CONDENSA_ERR_NULL;
    tb->td = arena.array<TensorDesc>(static_cast<size_t>(n_tensors) + 1);
    if (tb->td == nullptr) return CONDENSA_ERR_SIZE;
    tb->n_td = n_tensors + 1;
    u64 flat = 0, chunk = 0;
    for (int t = 0; t < n_tensors; ++t) {
        u64 n;
        if (!tensor_elems(tensors[t], &n)) return CONDENSA_ERR_SHAPE;
        if (n > 0 && tensors[t].w == nullptr) return CONDENSA_ERR_NULL;
        TensorDesc& d = tb->td[t];
        d.w = tensors[t].w;
        d.n = n;
        d.flat_start = flat;
        d.chunk_start = chunk;
        flat += n;
        if (flat > kMaxElems) return CONDENSA_ERR_SIZE;
        chunk += (n + kChunk - 1) / kChunk;
        if (n > 0 && !aligned16(d.w)) tb->vec = false;
    }
    TensorDesc& end = tb->td[n_tensors];
    end.flat_start = flat;
    end.chunk_start = chunk;
    tb->N = flat;
    tb->n_chunks = chunk;
    return CONDENSA_OK;
}

static condensa_status check_workspace(const void* ws, size_t bytes, const Layout& L) {
    if (ws == nullptr) return CONDENSA_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(ws) & 255u) return CONDENSA_ERR_WORKSPACE;
    if (bytes < L.total) return CONDENSA_ERR_WORKSPACE;
    return CONDENSA_OK;
}

static void init_slot(Slot* s, u64 n, u64 k, u32 path) {
    std::memset(s, 0, sizeof(Slot));
    s->n = n;
    s->k = k;
    s->path = path;
    if (k == 0) {
        s->state = kInactive;
        s->prefix = ~static_cast<u64>(0);
        s->remaining = 0;
        s->tie_end = 0;
    } else {
        s->state = kSelecting;
        s->prefix = 0;
        s->remaining = k;
        s->tie_end = n;
    }
}

// One density on the window path: the three rankings of the sample that bound (kRankHi, kRankLo) and estimate
// (kRankMid) the threshold of `main`.  Their ranks depend on the number of valid sample keys, which only the
// device knows, so the host passes the rule and the device turns it into a rank (sample_rank).
static void init_sample_slots(Slot* three, const Slot& main, int64_t margin16) {
    for (u32 i = 0; i < 3; ++i) {
        Slot& s = three[i];
        std::memset(&s, 0, sizeof(Slot));
        s.rank_rule = kRankHi + i;
        s.margin16 = static_cast<u32>(margin16);
        s.p = main.n ? static_cast<double>(main.k) / static_cast<double>(main.n) : 0.0;
        s.hi = 0x7FFFFFFFu;                                     // every valid sample key takes part
        s.state = main.state == kSelecting ? kSelecting : kDone;
        s.prefix = (s.rank_rule == kRankHi && s.state == kDone) ? 0x7FFFFFFFu : 0u;
    }
}

template <typename T>
static T* at(void* ws, size_t off) { return reinterpret_cast<T*>(static_cast<char*>(ws) + off); }

static unsigned fill_grid(u64 words) {
    u64 b = (words + kBlock - 1) / kBlock;
    if (b > 4096) b = 4096;
    if (b == 0) b = 1;
    return static_cast<unsigned>(b);
}

static condensa_status poke_upload(void* dst_dev, const char* src_host, size_t bytes, hipStream_t st);

// The image of a call's tables in its staging slot.
static UploadArgs fill_image(const StageImage& img, const Layout& L, void* ws, const Tables& tb, const OutDesc* out, size_t out_bytes,
                             const Slot* slots, size_t slot_bytes, const void* lists, size_t list_bytes) {
    const void* src[4] = {tb.td, out, slots, lists};
    const size_t bytes[4] = {static_cast<size_t>(tb.n_td) * sizeof(TensorDesc), out_bytes, slot_bytes, list_bytes};
    const size_t dst[4] = {L.td, L.out, L.slots, L.l_rank};
    UploadArgs up{};
    up.src = reinterpret_cast<const uint4*>(img.data());
    size_t at0 = 0;
    for (int i = 0; i < 4; ++i) {
        if (bytes[i]) std::memcpy(img.data() + at0, src[i], bytes[i]);
        at0 += bytes[i];
        up.dst[i] = at<uint4>(ws, dst[i]);
        up.end[i] = static_cast<u32>(at0 / 16);
    }
    up.done = img.done();
    up.ticket = img.ticket();
    return up;
}

// Workgroups of the launch that begins a call, beside the one that fetches the tables.
static u64 begin_blocks(u64 n_zero, u64 n_chunks) {
    const u64 words = n_zero > n_chunks ? n_zero : n_chunks;
    const u64 blocks = (words + 2 * kBeginThreads - 1) / (2 * kBeginThreads);
    return blocks > 512 ? 512 : (blocks ? blocks : 1);
}

static BeginTables begin_tables_args(const UploadArgs& up, const Layout& L, const Tables& tb, int n_tensors, void* ws) {
    BeginTables b{};
    b.up = up;
    b.zero = at<uint4>(ws, L.zero_begin);
    b.n_zero = L.zero_bytes / 16;
    b.chunk_map = at<u32>(ws, L.chunk_map);
    b.n_chunks = static_cast<u32>(tb.n_chunks);
    b.n_tensors = n_tensors;
    return b;
}

// What every call starts with: the tables [tensors | outputs | rankings] reach the front of the workspace, the
// counter and histogram region is cleared and the chunk -> tensor map is written.  One launch while the tables are
// small (kBeginTensors tensors, one staging slot), two beyond that.  Without a slot (`img`: a captured call, or none free) and for
// callers that cannot allocate (no `img`, but `fixed`: memory to build the image in) the tables travel as kernel
// arguments, which a graph copies.
static condensa_status begin_call(const Layout& L, const Tables& tb, int n_tensors, const OutDesc* out, size_t n_out,
                                  const Slot* slots, size_t n_slots, void* ws, hipStream_t st, StageImage* img,
                                  const void* lists = nullptr, size_t list_bytes = 0, char* fixed = nullptr) {
    const size_t td_bytes = static_cast<size_t>(tb.n_td) * sizeof(TensorDesc), out_bytes = n_out * sizeof(OutDesc),
                 slot_bytes = n_slots * sizeof(Slot);
    const u64 n_words = L.zero_bytes / 8;
    if (img) {
        const condensa_status rc = img->acquire(td_bytes + out_bytes + slot_bytes + list_bytes, st);    // each a multiple of 16 bytes
        if (rc != CONDENSA_OK) return rc;
    }
    if (img == nullptr || img->data() == nullptr) {
        std::vector<char> own;
        if (!fixed) { own.resize(L.upload_bytes); fixed = own.data(); }
        std::memcpy(fixed + L.td, tb.td, td_bytes);
        if (out_bytes) std::memcpy(fixed + L.out, out, out_bytes);
        if (slot_bytes) std::memcpy(fixed + L.slots, slots, slot_bytes);
        condensa_status rc = poke_upload(ws, fixed, L.upload_bytes, st);
        if (rc == CONDENSA_OK) rc = poke_upload(at<char>(ws, L.l_rank), static_cast<const char*>(lists), list_bytes, st);
        if (rc != CONDENSA_OK) return rc;
        hipLaunchKernelGGL(k_prepare, dim3(fill_grid(n_words)), dim3(kBlock), 0, st, at<u64>(ws, L.zero_begin), n_words,
                           at<TensorDesc>(ws, L.td), n_tensors, at<u32>(ws, L.chunk_map), tb.n_chunks,
                           static_cast<u64*>(nullptr), static_cast<u64>(0));
        CONDENSA_LAUNCH_CHECK();
        return CONDENSA_OK;
    }
    const UploadArgs up = fill_image(*img, L, ws, tb, out, out_bytes, slots, slot_bytes, lists, list_bytes);
    if (n_tensors <= kBeginTensors && td_bytes + out_bytes + slot_bytes + list_bytes <= kStageBytes) {
        BeginArgs b{};
        b.t = begin_tables_args(up, L, tb, n_tensors, ws);
        for (int t = 0; t <= n_tensors; ++t) b.chunk_start[t] = static_cast<u32>(tb.td[t].chunk_start);
        const u64 blocks = begin_blocks(b.t.n_zero, tb.n_chunks) + 1;
        img->launching(st);
        hipLaunchKernelGGL(k_begin, dim3(static_cast<unsigned>(blocks)), dim3(kBeginThreads), 0, st, b);
        CONDENSA_LAUNCH_CHECK();
        img->commit();
        return CONDENSA_OK;
    }
    const u32 up_blocks = (up.end[3] + 4 * kBlock - 1) / (4 * kBlock);
    img->launching(st);
    hipLaunchKernelGGL(k_upload, dim3(up_blocks ? up_blocks : 1), dim3(kBlock), 0, st, up);
    CONDENSA_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_prepare, dim3(fill_grid(n_words)), dim3(kBlock), 0, st, at<u64>(ws, L.zero_begin), n_words,
                       at<TensorDesc>(ws, L.td), n_tensors, at<u32>(ws, L.chunk_map), tb.n_chunks, img->done(), img->ticket());
    CONDENSA_LAUNCH_CHECK();
    img->commit();
    return CONDENSA_OK;
}

// Radix levels over the weights: 3 x (histogram sweep + bin search).
template <bool LC, bool VEC>
static condensa_status launch_radix_levels(const DataArgs& a, int n_slots, hipStream_t st, const Config& cfg) {
    if (a.n_chunks > 0) {
        // as the gated fallback of the window path these launches are (normally empty) resolve work
        PhaseTimer timer(a.only_failed ? CONDENSA_PHASE_RESOLVE : CONDENSA_PHASE_SWEEP, st, cfg);
        for (int level = 0; level < n_levels(31); ++level) {
            // Every workgroup flushes the non-zero bins of its LDS histograms (J of them past level 0) with
            // global atomics: few wide workgroups keep that flush small (level 0 of 20 M weights: 36 -> 19 us).
            const bool wide = !a.per_tensor;
            const unsigned threads = wide ? 1024 : kBlock;
            // measured: best of 128..1024 workgroups at 1.2 G weights; on 20 M weights (10 rankings) 256 x 1024
            // threads take 192 us per call against 221 (512 x 512), 275 (512 x 256) and 351 (1024 x 256)
            const u64 cap = wide ? 256 : 2048;
            const u64 per_iter = threads / kBlock;
            u64 blocks = (a.n_chunks + per_iter - 1) / per_iter;
            if (blocks > cap) blocks = cap;
            u64 cpb = (a.n_chunks + blocks - 1) / blocks;
            cpb = (cpb + per_iter - 1) / per_iter * per_iter;
            blocks = (a.n_chunks + cpb - 1) / cpb;
            const int nj = a.J < kSlotBatch ? a.J : kSlotBatch;
            const size_t lds = static_cast<size_t>(level == 0 ? kBins : nj * (1 << level_of(31, level).bits)) * sizeof(u32);
            hipLaunchKernelGGL((k_hist_data<LC, VEC>), dim3(static_cast<unsigned>(blocks)), dim3(threads), lds, st, a, level, cpb);
            CONDENSA_LAUNCH_CHECK();
            if (a.merged) continue;                            // the next kernel folds this level in itself
            hipLaunchKernelGGL(k_scan_level, dim3(n_slots), dim3(kBlock), 0, st, a.slots, a.hist0, a.histx, a.J, 31,
                               level, a.ctl, a.only_failed, &a.ctl->need_tie);
            CONDENSA_LAUNCH_CHECK();
        }
    }
    return CONDENSA_OK;
}

template <bool LC, bool VEC>
static condensa_status launch_ties_and_results(const DataArgs& a, int n_slots, int n_groups,
                                               condensa_select* results, hipStream_t st, const Config& cfg) {
    PhaseTimer timer(CONDENSA_PHASE_RESOLVE, st, cfg);
    if (a.n_chunks > 0) {
        // merged form: every workgroup first folds in the last level for each ranking, so fewer of them
        const u64 tie_cap = a.merged ? 1024 : 4096;
        const unsigned tie_blocks = static_cast<unsigned>(a.n_chunks < tie_cap ? a.n_chunks : tie_cap);
        hipLaunchKernelGGL((k_tie_count<LC, VEC>), dim3(tie_blocks), dim3(kBlock), 0, st, a);
        CONDENSA_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL((k_tie_locate<LC, VEC>), dim3(n_slots), dim3(kBlock), 0, st, a, results, n_groups);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}

template <bool LC, bool VEC>
static condensa_status run_selection(DataArgs a, const Layout& L, void* ws, bool use_window, int n_slots,
                                     int n_groups, condensa_select* results, hipStream_t st, const Config& cfg,
                                     const FusedRequest* fused = nullptr) {
    condensa_status rc;
    if (use_window) {
        rc = a.J == 1 ? launch_window_path_single<LC, VEC>(a, L, ws, st, cfg, fused)
                      : launch_window_path<LC, VEC>(a, L, ws, st, cfg);
        if (rc != CONDENSA_OK) return rc;
        a.only_failed = 1;
    }
    rc = launch_radix_levels<LC, VEC>(a, n_slots, st, cfg);
    if (rc != CONDENSA_OK) return rc;
    return launch_ties_and_results<LC, VEC>(a, n_slots, n_groups, results, st, cfg);
}

// The listed windows (k_listed.h).  With `write` the one pass over the weights writes the outputs; without it (an
// output that overwrites its input, or two sweeps asked for) the caller's apply sweep follows.
struct ListRequest {
    const OutDesc* out;    // device output table
    bool vec_out;          // every output pointer allows 128-bit accesses
    bool pq;
    bool write;
    u64* nnz_out;
    bool wide;             // masks only, each 16-byte aligned
};

// What a call's populations ask for.
struct ListShape {
    u32 groups = 0;        // sampling workgroups
    bool bounds = false;   // some population has several
    bool lone = true;      // no population is larger than list_lone
    u32 fewer = kFewerNone;
};

// Host tables of the path: one ListRank per ranking, then (PER_TENSOR) the tensor of every sampling workgroup.
static size_t build_list_table(const Tables& tb, const Layout& L, int n_tensors, int J, bool per_tensor, bool lc, const Config& cfg,
                               std::vector<char>* table, ListShape* shape) {
    const size_t n_groups = per_tensor ? static_cast<size_t>(n_tensors) : 1;
    std::vector<u32> group_of;
    table->assign(n_groups * J * sizeof(ListRank), 0);
    ListRank* rk = reinterpret_cast<ListRank*>(table->data());
    u64 base = 0;
    u32 first = 0;
    *shape = ListShape{};
    u32 most = static_cast<u32>(kListMaxW);                // sampling workgroups of a population
    auto groups_of = [&](u64 n) {
        const u32 asked = list_groups(n, J, per_tensor, cfg);
        return per_tensor && cfg[CONDENSA_OPT_SAMPLE_LOG2] <= 0 ? list_fewer_groups(asked, most) : asked;
    };
    for (u64 asked; per_tensor && most > 32 && cfg[CONDENSA_OPT_SAMPLE_LOG2] <= 0; most /= 2) {
        asked = 0;
        for (size_t g = 0; g < n_groups; ++g) asked += groups_of(tb.td[g].n);
        if (asked <= kSampleResident) break;
    }
    auto segments_of = [&](u64 n) { return list_segments(n, list_wave_elems(tb.N, J, lc), L.l_max_segs); };
    // twice the room for populations of up to 2^23 elements that get fewer, where the workspace has it (list_units)
    auto room_of = [&](u64 n, u32 times) {
        return n ? (times == 2 && n <= (1u << 23) && list_fewer(groups_of(n), n) ? 2 : 1) * list_entries(n, segments_of(n), cfg) : 0;
    };
    u64 room = 0;
    for (size_t g = 0; per_tensor && g < n_groups; ++g) room += static_cast<u64>(J) * room_of(tb.td[g].n, 2);
    const u32 times = per_tensor && room <= L.cand_cap ? 2 : 1;
    shape->fewer = !per_tensor || cfg[CONDENSA_OPT_SAMPLE_LOG2] > 0 ? kFewerNone : (times == 2 ? kFewerLong : kFewerDeep);
    for (size_t g = 0; g < n_groups; ++g) {
        const u64 n = per_tensor ? tb.td[g].n : tb.N;
        const u32 w = groups_of(n), segs = segments_of(n);
        for (int j = 0; j < J; ++j) {
            ListRank& r = rk[g * J + j];
            const u64 entries = room_of(n, times);
            r.base = base;
            r.n_segs = segs;
            r.seg_cap = static_cast<u32>(entries / segs);
            r.group0 = first;
            r.n_groups = w;
            base += entries;
        }
        if (per_tensor) group_of.insert(group_of.end(), w, static_cast<u32>(g));
        if (w > 1) shape->bounds = true;
        if (n > list_lone(J, per_tensor)) shape->lone = false;
        first += w;
    }
    shape->groups = first;
    if (per_tensor) {
        const size_t at0 = table->size();
        table->resize(align_up(at0 + group_of.size() * sizeof(u32), 16), 0);
        std::memcpy(table->data() + at0, group_of.data(), group_of.size() * sizeof(u32));
    }
    return table->size();
}

static ListArgs list_args(const Layout& L, void* ws, u64 N, int n_slots, const ListShape& shape, const ListRequest& rq, const Config& cfg) {
    ListArgs w{};
    w.rank = at<ListRank>(ws, L.l_rank);
    w.group_of = reinterpret_cast<const u32*>(w.rank + n_slots);
    w.local = at<u64>(ws, L.l_local);
    w.n_local = shape.groups;
    w.win = at<ListWin>(ws, L.l_win);
    w.sorted = at<ListSorted>(ws, L.l_sorted);
    w.max_segs = L.l_max_segs;
    w.n_rankings = n_slots;
    w.hist = at<u32>(ws, L.l_hist);
    w.hist_copies = list_hist_copies(n_slots);
    w.uneven_copies = list_uneven_copies(n_slots);
    w.count_in_sweep = !shape.lone && n_slots == 1 ? 1 : 0;
    w.arrived = at<u32>(ws, L.l_post);
    w.ended = w.arrived + kListLine;
    w.picked = at<u64>(ws, L.l_posted);
    w.verdict = w.picked + list_posted(N);
    w.range = reinterpret_cast<u32*>(w.verdict + list_walkers(N));
    w.gathered = at<u32>(ws, L.l_gathered);
    w.bin_want = at<u32>(ws, L.l_want);
    w.gkey = at<u32>(ws, L.l_gkey);
    w.gidx = at<u32>(ws, L.l_gidx);
    w.gather_cap = L.l_gather_cap;
    // workgroups that walk each list (several rankings): about a thousand in all, up to 256 for one ranking (134 M weights want them all).  At least 64 where
    // the rankings share a population (four densities of 20 M weights 76.3 us with 38, 73.6 with 64, 73.8 with 100; ten 107.5, 105.0 and 104.9, the same as 64
    // from 0.4 to 6 M weights); 32 where each has its own (16 of 2^20 weights 64.0 us with 32, 64.8 with 64; 17 layers of VGG-19 72.6 with 38 and with 60)
    const u64 least = L.n_groups > 1 ? 32 : 64;
    const u64 by_size = (N >> 19) < least ? least : ((N >> 19) > 256 ? 256 : N >> 19);
    const u64 share = n_slots >= 1024 ? 1 : 1024 / static_cast<u64>(n_slots);
    w.parts = static_cast<u32>(by_size < share ? by_size : share);
    w.cnt = at<u64>(ws, L.l_cnt);
    w.nnz = at<u32>(ws, L.l_nnz);
    w.key = at<u32>(ws, L.l_key);
    w.idx = at<u32>(ws, L.l_idx);
    w.gmax = at<u32>(ws, L.l_gmax);
    w.gmaxc = w.gmax + n_slots;
    w.fb = at<FallbackCtl>(ws, L.l_fb);
    w.special = at<u32>(ws, L.l_special);
    w.fb_above = w.special + n_slots;
    w.state = at<ListState>(ws, L.l_state);
    w.open_of = at<u32>(ws, L.l_masks);
    w.tie_of = w.open_of + L.n_groups;
    w.apply_of = w.tie_of + L.n_groups;
    w.fb_hist = at<u32>(ws, L.l_fb_hist);
    w.fb_bins = L.l_fb_bins;
    w.meet = at<u32>(ws, L.l_meet);
    w.cand_shift = static_cast<int>(cfg[CONDENSA_OPT_CAND_SHIFT]);
    w.out = rq.out;
    w.nnz_out = rq.nnz_out;
    w.margin16 = static_cast<int>(cfg[CONDENSA_OPT_WINDOW_MARGIN]);
    w.write = rq.write ? 1 : 0;
    w.force = t_force;
    w.fewer = shape.fewer;
    return w;
}

// Tag of a call's words in ListArgs::local: another one for each of 2^32 calls, and none that a workspace is likely to hold.  The
// mixing is the 32-bit finalizer of MurmurHash3 (A. Appleby, public domain), with its constants.
static u32 call_tag(u32 call) {
    u32 x = call + 0x9E3779B9u;
    x = (x ^ (x >> 16)) * 0x85EBCA6Bu;
    x = (x ^ (x >> 13)) * 0xC2B2AE35u;
    return x ^ (x >> 16);
}

static u32 next_tag() {
    static std::atomic<u32> calls{0};
    return call_tag(calls.fetch_add(1, std::memory_order_relaxed));
}

// Begins the call, takes the sample and bounds the windows in one launch; false when the call is not of that form.
template <bool LC, bool VEC>
static condensa_status begin_and_sample(const Layout& L, const Tables& tb, int n_tensors, const OutDesc* out, size_t n_out, const Slot* slots,
                                        const double* densities, int J, bool per_tensor, float mu, void* ws, hipStream_t st,
                                        const std::vector<char>& lists, const ListShape& shape, const ListRequest& rq, const Config& cfg, StageImage* img, bool* begun) {
    *begun = false;
    const u32 groups = shape.groups;
    const size_t td_bytes = static_cast<size_t>(tb.n_td) * sizeof(TensorDesc), out_bytes = n_out * sizeof(OutDesc),
                 slot_bytes = static_cast<size_t>(L.n_slots) * sizeof(Slot);
    if (n_tensors > kBeginSampleTensors || groups > 0xFFFFu || td_bytes + out_bytes + slot_bytes + lists.size() > kStageBytes) return CONDENSA_OK;
    const condensa_status rc = img->acquire(td_bytes + out_bytes + slot_bytes + lists.size(), st);
    if (rc != CONDENSA_OK || img->data() == nullptr) return rc;
    PhaseTimer timer(CONDENSA_PHASE_SAMPLE, st, cfg);
    BeginSampleArgs b{};
    b.up = fill_image(*img, L, ws, tb, out, out_bytes, slots, slot_bytes, lists.data(), lists.size());
    b.zero = at<uint4>(ws, L.zero_begin);
    b.n_zero = L.zero_bytes / 16;
    b.chunk_map = at<u32>(ws, L.chunk_map);
    b.n_chunks = static_cast<u32>(tb.n_chunks);
    b.n_tensors = n_tensors;
    b.groups = groups;
    b.J = J;
    b.mu = mu;
    b.N = tb.N;
    b.per_tensor = per_tensor ? 1 : 0;
    for (int j = 0; j < J; ++j) b.density[j] = densities[j];
    const ListRank* rk = reinterpret_cast<const ListRank*>(lists.data());
    for (int t = 0; per_tensor && t < n_tensors; ++t) b.group0[t] = static_cast<u16>(rk[static_cast<size_t>(t) * J].group0);
    b.group0[per_tensor ? n_tensors : 0] = static_cast<u16>(groups);
    for (int t = 0; t < n_tensors; ++t) {
        b.w[t] = tb.td[t].w;
        b.lam[t] = tb.td[t].lam;
        b.n[t] = static_cast<u32>(tb.td[t].n);
    }
    for (int t = 0; t <= n_tensors; ++t) b.chunk_start[t] = static_cast<u32>(tb.td[t].chunk_start);
    b.fillers = static_cast<u32>(begin_blocks(b.n_zero, tb.n_chunks));
    const u32 bounds = shape.bounds ? (per_tensor ? static_cast<u32>(n_tensors) : 1u) : 0u;
    ListArgs w = list_args(L, ws, tb.N, L.n_slots, shape, rq, cfg);
    w.tag = next_tag();
    img->launching(st);
    const dim3 grid(1 + groups + b.fillers + bounds);
    if (L.l_gather_cap > kListGather) hipLaunchKernelGGL((k_begin_sample<LC, VEC, true>), grid, dim3(kListThreads), sample_lds(J), st, b, w);
    else                              hipLaunchKernelGGL((k_begin_sample<LC, VEC, false>), grid, dim3(kListThreads), sample_lds(J), st, b, w);
    CONDENSA_LAUNCH_CHECK();
    img->commit();
    *begun = true;
    return CONDENSA_OK;
}

template <bool LC, bool VEC>
static condensa_status launch_listed(const DataArgs& a, const Layout& L, void* ws, const ListShape& shape, int n_slots, int n_groups,
                                     condensa_select* results, const ListRequest& rq, bool sampled, hipStream_t st, const Config& cfg) {
    ListArgs w = list_args(L, ws, a.N, n_slots, shape, rq, cfg);
    const bool vec = VEC && rq.vec_out;
    if (!sampled) {
        PhaseTimer timer(CONDENSA_PHASE_SAMPLE, st, cfg);
        hipLaunchKernelGGL((k_list_sample<LC, VEC>), dim3(shape.groups), dim3(kListThreads), sample_lds(a.J), st, a, w);
        CONDENSA_LAUNCH_CHECK();
        if (shape.bounds) {
            hipLaunchKernelGGL(k_list_bounds, dim3(static_cast<unsigned>(n_groups)), dim3(kBoundsThreads), 0, st, a, w);
            CONDENSA_LAUNCH_CHECK();
        }
    }
    {
        PhaseTimer timer(CONDENSA_PHASE_SWEEP, st, cfg);
        constexpr int Q = LC ? kFusedQuadsLC : kFusedQuadsPrune;
        const dim3 grid(static_cast<unsigned>(a.n_chunks * (kChunk / (256 * Q))));
        if constexpr (LC) {
            if (rq.pq && vec)  hipLaunchKernelGGL((k_list_sweep<true, true, Q, true>), grid, dim3(64), 0, st, a, w);
            else if (rq.pq)    hipLaunchKernelGGL((k_list_sweep<true, false, Q, true>), grid, dim3(64), 0, st, a, w);
            else if (vec)      hipLaunchKernelGGL((k_list_sweep<true, true, Q, false>), grid, dim3(64), 0, st, a, w);
            else               hipLaunchKernelGGL((k_list_sweep<true, false, Q, false>), grid, dim3(64), 0, st, a, w);
        } else if (a.J == 1) {
            if (vec) hipLaunchKernelGGL((k_list_sweep<false, true, Q, false>), grid, dim3(64), 0, st, a, w);
            else     hipLaunchKernelGGL((k_list_sweep<false, false, Q, false>), grid, dim3(64), 0, st, a, w);
        } else {
            const int quads = list_multi_quads(a.N);
            const dim3 gm(static_cast<unsigned>(a.n_chunks * (kChunk / (256 * static_cast<unsigned>(quads)))));
            constexpr int QM = kListMultiQuads;
            if (quads == 1 && vec)  hipLaunchKernelGGL((k_list_sweep_multi<true, false, 1>), gm, dim3(64), 0, st, a, w);
            else if (quads == 1)    hipLaunchKernelGGL((k_list_sweep_multi<false, false, 1>), gm, dim3(64), 0, st, a, w);
            else if (vec && rq.wide) hipLaunchKernelGGL((k_list_sweep_multi<true, true, QM>), gm, dim3(64), 0, st, a, w);
            else if (vec)           hipLaunchKernelGGL((k_list_sweep_multi<true, false, QM>), gm, dim3(64), 0, st, a, w);
            else                    hipLaunchKernelGGL((k_list_sweep_multi<false, false, QM>), gm, dim3(64), 0, st, a, w);
        }
        CONDENSA_LAUNCH_CHECK();
    }
    PhaseTimer timer(CONDENSA_PHASE_RESOLVE, st, cfg);
    const dim3 walk(static_cast<unsigned>(n_slots) * w.parts), fb(kSettleGrid);
    const int vo = rq.vec_out ? 1 : 0;
    if (shape.lone) {
        const dim3 fin(static_cast<unsigned>(n_slots));
        if (LC && rq.pq) hipLaunchKernelGGL((k_list_finish<LC, VEC, LC>), fin, dim3(kListThreads), 0, st, a, w, results, n_groups, vo);
        else             hipLaunchKernelGGL((k_list_finish<LC, VEC, false>), fin, dim3(kListThreads), 0, st, a, w, results, n_groups, vo);
        CONDENSA_LAUNCH_CHECK();
        return CONDENSA_OK;
    }
    if (n_slots == 1) {
        for (int late = 0; late <= ((t_force & kForceLate) ? 1 : 0); ++late) {
            const bool is_long = list_long(a.N);
            if (is_long && LC && rq.pq) hipLaunchKernelGGL((k_list_resolve<LC, VEC, LC, true>), fb, dim3(kSettleThreads), 0, st, a, w, results, vo);
            else if (is_long)           hipLaunchKernelGGL((k_list_resolve<LC, VEC, false, true>), fb, dim3(kSettleThreads), 0, st, a, w, results, vo);
            else if (LC && rq.pq)       hipLaunchKernelGGL((k_list_resolve<LC, VEC, LC, false>), fb, dim3(kSettleThreads), 0, st, a, w, results, vo);
            else                        hipLaunchKernelGGL((k_list_resolve<LC, VEC, false, false>), fb, dim3(kSettleThreads), 0, st, a, w, results, vo);
            CONDENSA_LAUNCH_CHECK();
        }
        return CONDENSA_OK;
    }
    if constexpr (!LC) {                                   // (an L-C step has one ranking)
        hipLaunchKernelGGL(k_list_hist, walk, dim3(kBlock), 0, st, w);
        CONDENSA_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_list_gather, walk, dim3(kBlock), 0, st, a, w);
        CONDENSA_LAUNCH_CHECK();
        hipLaunchKernelGGL((k_list_settle<VEC>), fb, dim3(kSettleThreads), 0, st, a, w, results, n_groups, vo);
        CONDENSA_LAUNCH_CHECK();
    }
    return CONDENSA_OK;
}

}  // namespace condensa

namespace condensa {

// ---- static scratch for callers that cannot allocate ---------------------------------------------------
// One array per device, resident until the process ends.  Host code never uses the array's name as an
// address: scratch_for_current_device() asks the runtime for the device address once per device.

constexpr size_t kScratchBytes = static_cast<size_t>(2) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;
}  // namespace

static condensa_status scratch_for_current_device(void** out) {
    int dev = -1;
    CONDENSA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return CONDENSA_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        CONDENSA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (p == nullptr) return CONDENSA_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return CONDENSA_OK;
}

// Writes host words into device memory as kernel arguments: no staging buffer, nothing to allocate.
struct PokeWords { u64 w[448]; };
__global__ __launch_bounds__(kBlock) void k_poke(u64* dst, PokeWords src, u32 n) {
    for (u32 i = threadIdx.x; i < n; i += kBlock) dst[i] = src.w[i];
}

static condensa_status poke_upload(void* dst_dev, const char* src_host, size_t bytes, hipStream_t st) {
    constexpr size_t kPiece = sizeof(PokeWords);
    for (size_t off = 0; off < bytes; off += kPiece) {
        const size_t n = bytes - off < kPiece ? bytes - off : kPiece;      // bytes is a multiple of 16
        PokeWords pw;
        std::memcpy(pw.w, src_host + off, n);
        hipLaunchKernelGGL(k_poke, dim3(1), dim3(kBlock), 0, st, reinterpret_cast<u64*>(static_cast<char*>(dst_dev) + off),
                           pw, static_cast<u32>(n / 8));
        CONDENSA_LAUNCH_CHECK();
    }
    return CONDENSA_OK;
}

// condensa_prune and its allocation-free form share everything but where the host tables live, how they
// reach the device and where the workspace comes from.
static condensa_status prune_impl(const condensa_tensor* tensors, int n_tensors, const double* densities,
                                  int n_densities, int scope, float* const* theta, uint16_t* const* theta_f16,
                                  uint8_t* const* mask, condensa_select* results_dev, void* workspace_dev,
                                  size_t workspace_bytes, void* stream, const Config& given, HostArena& arena,
                                  bool no_alloc) {
    if (n_densities < 1 || n_densities > CONDENSA_MAX_DENSITIES) return CONDENSA_ERR_SIZE;
    if (densities == nullptr || results_dev == nullptr) return CONDENSA_ERR_NULL;
    if (scope != CONDENSA_SCOPE_GLOBAL && scope != CONDENSA_SCOPE_PER_TENSOR) return CONDENSA_ERR_ARG;
    for (int j = 0; j < n_densities; ++j)
        if (!density_ok(densities[j])) return CONDENSA_ERR_DENSITY;
    Tables tb;
    condensa_status rc = build_tensor_table(tensors, n_tensors, &tb, arena);
    if (rc != CONDENSA_OK) return rc;
    const int J = n_densities;
    const bool per_tensor = (scope == CONDENSA_SCOPE_PER_TENSOR);
    if (per_tensor && n_tensors == 0) return CONDENSA_OK;
    // the allocation-free form keeps to the radix levels, whose workspace is small whatever the input
    Config cfg = given;
    Layout L = make_layout(CONDENSA_OP_PRUNE, tb.N, 0, n_tensors, J, scope, cfg, no_alloc);

    // output table, overlap and alignment checks
    const bool any_out = theta || theta_f16 || mask;
    const size_t n_out = static_cast<size_t>(J) * (n_tensors > 0 ? n_tensors : 1);
    OutDesc* out = arena.array<OutDesc>(n_out);
    ByteRange* ranges = arena.array<ByteRange>(static_cast<size_t>(n_tensors) * (1 + 3 * J) + 2);
    if (!out || !ranges) return CONDENSA_ERR_SIZE;
    size_t n_ranges = 0;
    bool vec = tb.vec, masks_wide = true;
    bool in_place_any = false;
    for (int t = 0; t < n_tensors; ++t) {
        const u64 n = tb.td[t].n;
        if (n == 0) continue;
        bool in_place = false;
        for (int j = 0; j < J; ++j) {
            const size_t i = static_cast<size_t>(j) * n_tensors + t;
            OutDesc& o = out[i];
            o.theta = theta ? theta[i] : nullptr;
            o.theta16 = theta_f16 ? theta_f16[i] : nullptr;
            o.mask = mask ? mask[i] : nullptr;
            if (o.theta == tb.td[t].w) {                    // in place: one density only
                if (J > 1) return CONDENSA_ERR_ARG;
                in_place = true;
            } else {
                ranges[n_ranges++] = byte_range(o.theta, n * 4, true);
            }
            ranges[n_ranges++] = byte_range(o.theta16, n * 2, true);
            ranges[n_ranges++] = byte_range(o.mask, n, true);
            if (o.theta && !aligned16(o.theta)) vec = false;
            if (o.theta16 && (reinterpret_cast<uintptr_t>(o.theta16) & 7u)) vec = false;
            if (o.mask && (reinterpret_cast<uintptr_t>(o.mask) & 3u)) vec = false;
            if (!aligned16(o.mask)) masks_wide = false;
        }
        ranges[n_ranges++] = byte_range(tb.td[t].w, n * 4, in_place);
        in_place_any = in_place_any || in_place;
    }
    if (J == 1 && !per_tensor && (!any_out || in_place_any || cfg[CONDENSA_OPT_FUSED_SWEEP] != 0))
        prefer_window_for_two_sweeps(CONDENSA_OP_PRUNE, tb.N, n_tensors, workspace_bytes, &cfg, &L);
    fewer_gathered_where_short(CONDENSA_OP_PRUNE, tb.N, n_tensors, J, scope, workspace_bytes, cfg, &L);
    ranges[n_ranges++] = byte_range(workspace_dev, workspace_bytes < L.total ? workspace_bytes : L.total, true);
    ranges[n_ranges++] = byte_range(results_dev, static_cast<u64>(L.n_slots) * sizeof(condensa_select), true);
    if (ranges_conflict(ranges, n_ranges)) return CONDENSA_ERR_ARG;
    rc = check_workspace(workspace_dev, workspace_bytes, L);
    if (rc != CONDENSA_OK) return no_alloc ? CONDENSA_ERR_SIZE : rc;

    const bool window = !no_alloc && want_window(tb.N, n_tensors, per_tensor, J, cfg);
    Slot* slots = arena.array<Slot>(static_cast<size_t>(L.n_slots) + 3);
    char* fixed = no_alloc ? arena.array<char>(L.upload_bytes) : nullptr;
    if (!slots || (no_alloc && !fixed)) return CONDENSA_ERR_SIZE;
    for (int g = 0; g < L.n_groups; ++g)
        for (int j = 0; j < J; ++j) {
            const u64 n = per_tensor ? tb.td[g].n : tb.N;
            init_slot(&slots[static_cast<size_t>(g) * J + j], n, kept_count(densities[j], n), window || L.listed ? 2u : 1u);
        }
    const size_t n_up_slots = static_cast<size_t>(L.n_slots) + ((window && J == 1) ? 3 : 0);
    if (window && J == 1) init_sample_slots(slots + L.n_slots, slots[0], cfg[CONDENSA_OPT_WINDOW_MARGIN]);

    hipStream_t st = static_cast<hipStream_t>(stream);
    std::vector<char> lists;
    ListShape list_shape;
    const size_t list_bytes = L.listed ? build_list_table(tb, L, n_tensors, J, per_tensor, false, cfg, &lists, &list_shape) : 0;
    const OutDesc* od = at<OutDesc>(workspace_dev, L.out);
    const bool listed_write = L.listed && any_out && !in_place_any && cfg[CONDENSA_OPT_FUSED_SWEEP] == 0;
    const ListRequest rq{od, vec, false, listed_write, nullptr, masks_wide && !theta && !theta_f16};
    bool sampled = false;
    StageImage img;
    if (L.listed)
        rc = tb.vec ? begin_and_sample<false, true>(L, tb, n_tensors, out, n_out, slots, densities, J, per_tensor, 0.0f, workspace_dev, st, lists, list_shape, rq, cfg, &img, &sampled)
                    : begin_and_sample<false, false>(L, tb, n_tensors, out, n_out, slots, densities, J, per_tensor, 0.0f, workspace_dev, st, lists, list_shape, rq, cfg, &img, &sampled);
    if (rc == CONDENSA_OK && !sampled)
        rc = begin_call(L, tb, n_tensors, out, n_out, slots, n_up_slots, workspace_dev, st, no_alloc ? nullptr : &img, lists.data(), list_bytes, fixed);
    if (rc != CONDENSA_OK) return rc;

    DataArgs a{};
    a.td = at<TensorDesc>(workspace_dev, L.td);
    a.slots = at<Slot>(workspace_dev, L.slots);
    a.hist0 = at<u64>(workspace_dev, L.hist0);
    a.histx = at<u64>(workspace_dev, L.histx);
    a.coarse = at<u64>(workspace_dev, L.histc);
    a.tiecnt = at<u32>(workspace_dev, L.tiecnt);
    a.tiehit = at<u32>(workspace_dev, L.tiehit);
    if (L.tl_key) {
        a.tl_cnt = at<u64>(workspace_dev, L.tl_cnt);
        a.tl_key = at<u32>(workspace_dev, L.tl_key);
        a.tl_idx = at<u64>(workspace_dev, L.tl_idx);
    }
    a.ctl = at<Control>(workspace_dev, L.ctl);
    a.chunk_map = at<u32>(workspace_dev, L.chunk_map);
    a.n_chunks = tb.n_chunks;
    a.N = tb.N;
    a.n_tensors = n_tensors;
    a.J = J;
    a.per_tensor = per_tensor ? 1 : 0;
    a.only_failed = 0;
    a.streaming = (tb.N * 4u >= (static_cast<u64>(512) << 20)) ? 1 : 0;            // well beyond the 256 MB last-level cache
    a.mu = 0.0f;
    a.merged = per_tensor ? 0 : 1;

    if (L.listed) {
        rc = tb.vec ? launch_listed<false, true>(a, L, workspace_dev, list_shape, L.n_slots, L.n_groups, results_dev, rq, sampled, st, cfg)
                    : launch_listed<false, false>(a, L, workspace_dev, list_shape, L.n_slots, L.n_groups, results_dev, rq, sampled, st, cfg);
        if (rc != CONDENSA_OK || listed_write) return rc;
    }
    // One density on the window path: selection and apply share one sweep unless theta overwrites the weights.
    const bool fuse = window && J == 1 && any_out && tb.n_chunks > 0 && slots[0].k > 0 && !in_place_any &&
                      cfg[CONDENSA_OPT_FUSED_SWEEP] == 0;
    WindowArgs wargs{};
    FusedRequest fr{od, vec, false, &wargs};
    if (!L.listed)
        rc = tb.vec ? run_selection<false, true>(a, L, workspace_dev, window, L.n_slots, L.n_groups, results_dev, st, cfg, fuse ? &fr : nullptr)
                    : run_selection<false, false>(a, L, workspace_dev, window, L.n_slots, L.n_groups, results_dev, st, cfg, fuse ? &fr : nullptr);
    if (rc != CONDENSA_OK) return rc;

    if (fuse) {
        PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
        hipLaunchKernelGGL((k_window_fixup<false, false>), dim3(wargs.n_segs * kFixupParts), dim3(kBlock), 0, st, a, wargs);
        CONDENSA_LAUNCH_CHECK();
        const u64 n_tiles = tb.n_chunks * kSubPerChunk;
        const unsigned grid = static_cast<unsigned>(n_tiles < 4096 ? n_tiles : 4096);
        if (vec) hipLaunchKernelGGL((k_prune_apply_gated<true>), dim3(grid), dim3(kBlock), 0, st, a, od, n_tiles);
        else     hipLaunchKernelGGL((k_prune_apply_gated<false>), dim3(grid), dim3(kBlock), 0, st, a, od, n_tiles);
        CONDENSA_LAUNCH_CHECK();
    } else if (any_out && tb.n_chunks > 0) {
        PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
        if (vec) hipLaunchKernelGGL((k_prune_apply<true>), dim3(static_cast<unsigned>(tb.n_chunks * kSubPerChunk)), dim3(kBlock), 0, st, a, od);
        else     hipLaunchKernelGGL((k_prune_apply<false>), dim3(static_cast<unsigned>(tb.n_chunks * kSubPerChunk)), dim3(kBlock), 0, st, a, od);
        CONDENSA_LAUNCH_CHECK();
    }
    return CONDENSA_OK;
}

}  // namespace condensa

using namespace condensa;

// =====================================================================================================

extern "C" {

condensa_status condensa_config_init(condensa_config* config) {
    if (config == nullptr) return CONDENSA_ERR_NULL;
    Config c;
    resolve_config(nullptr, &c);
    config->select_path = static_cast<int32_t>(c[CONDENSA_OPT_SELECT_PATH]);
    config->sample_log2 = static_cast<int32_t>(c[CONDENSA_OPT_SAMPLE_LOG2]);
    config->window_margin = static_cast<int32_t>(c[CONDENSA_OPT_WINDOW_MARGIN]);
    config->cand_shift = static_cast<int32_t>(c[CONDENSA_OPT_CAND_SHIFT]);
    config->profile = static_cast<int32_t>(c[CONDENSA_OPT_PROFILE]);
    config->apply_threads = static_cast<int32_t>(c[CONDENSA_OPT_APPLY_THREADS]);
    config->fused_sweep = static_cast<int32_t>(c[CONDENSA_OPT_FUSED_SWEEP]);
    config->reserved = 0;
    return CONDENSA_OK;
}

size_t condensa_workspace_bytes(int op, uint64_t total_elems, uint64_t n_structures, int n_tensors,
                                int n_densities, int scope, const condensa_config* config) {
    if (op < CONDENSA_OP_PRUNE || op > CONDENSA_OP_LC_SGD_STEP) return 0;
    if (op == CONDENSA_OP_QUANTIZE) return 0;
    if (n_tensors < 0 || n_tensors > CONDENSA_MAX_TENSORS) return 0;
    if (n_densities < 1 || n_densities > CONDENSA_MAX_DENSITIES) return 0;
    if (scope != CONDENSA_SCOPE_GLOBAL && scope != CONDENSA_SCOPE_PER_TENSOR) return 0;
    if (total_elems > kMaxElems || n_structures > total_elems) return 0;
    Config cfg;
    if (resolve_config(config, &cfg) != CONDENSA_OK) return 0;
    const size_t total = make_layout(op, total_elems, n_structures, n_tensors, n_densities, scope, cfg).total;
    // Large calls that choose their path answer for the sampled window too, which needs more (1.2 G weights: 766 MB, listed 205): two sweeps take
    // it by themselves, and who has asked without a configuration can ask for that path with the same workspace.  Smaller ones never could.
    if (cfg[CONDENSA_OPT_SELECT_PATH] != 0 || n_densities != 1 || scope != CONDENSA_SCOPE_GLOBAL || (op != CONDENSA_OP_PRUNE && op != CONDENSA_OP_LC_STEP) ||
        total_elems < (static_cast<u64>(3) << 26)) return total;
    cfg.v[CONDENSA_OPT_SELECT_PATH] = 2;
    const size_t window = make_layout(op, total_elems, n_structures, n_tensors, n_densities, scope, cfg).total;
    return window > total ? window : total;
}

condensa_status condensa_prune(const condensa_tensor* tensors, int n_tensors, const double* densities,
                               int n_densities, int scope, float* const* theta, uint16_t* const* theta_f16,
                               uint8_t* const* mask, condensa_select* results_dev, void* workspace_dev,
                               size_t workspace_bytes, void* stream, const condensa_config* config) {
    Config cfg;
    const condensa_status rc = resolve_config(config, &cfg);
    if (rc != CONDENSA_OK) return rc;
    HostArena arena;
    return prune_impl(tensors, n_tensors, densities, n_densities, scope, theta, theta_f16, mask, results_dev,
                      workspace_dev, workspace_bytes, stream, cfg, arena, false);
}

condensa_status condensa_prune_static(const condensa_tensor* tensors, int n_tensors, const double* densities,
                                      int n_densities, float* const* theta, uint16_t* const* theta_f16,
                                      uint8_t* const* mask, condensa_select* results_dev, void* stream) {
    if (n_tensors < 0 || n_tensors > CONDENSA_STATIC_MAX_TENSORS) return CONDENSA_ERR_SIZE;
    if (n_densities < 1 || n_densities > CONDENSA_STATIC_MAX_DENSITIES) return CONDENSA_ERR_SIZE;
    if (n_tensors > 0 && tensors == nullptr) return CONDENSA_ERR_NULL;
    u64 total = 0;
    for (int t = 0; t < n_tensors; ++t) {
        u64 n;
        if (!tensor_elems(tensors[t], &n)) return CONDENSA_ERR_SHAPE;
        total += n;
        if (total > CONDENSA_STATIC_MAX_ELEMS) return CONDENSA_ERR_SIZE;
    }
    // built-in settings: nothing of the process-wide defaults applies (no event is created for phase timing)
    Config cfg{};
    cfg.v[CONDENSA_OPT_SELECT_PATH] = 1;
    cfg.v[CONDENSA_OPT_WINDOW_MARGIN] = 80;
    void* ws = nullptr;
    const condensa_status rc = scratch_for_current_device(&ws);
    if (rc != CONDENSA_OK) return rc;
    // host tables on this stack frame: tensor table, output table, rankings, their upload image, byte ranges
    constexpr size_t kHostBytes =
        static_cast<size_t>(CONDENSA_STATIC_MAX_TENSORS + 1) * sizeof(TensorDesc) * 2 +
        static_cast<size_t>(CONDENSA_STATIC_MAX_TENSORS) * CONDENSA_STATIC_MAX_DENSITIES * sizeof(OutDesc) * 2 +
        static_cast<size_t>(CONDENSA_STATIC_MAX_DENSITIES + 2 * kMaxJ) * sizeof(Slot) * 2 +
        (static_cast<size_t>(CONDENSA_STATIC_MAX_TENSORS) * (1 + 3 * CONDENSA_STATIC_MAX_DENSITIES) + 2) * sizeof(ByteRange) +
        4096;
    alignas(64) char host[kHostBytes];
    HostArena arena(host, sizeof(host));
    return prune_impl(tensors, n_tensors, densities, n_densities, CONDENSA_SCOPE_GLOBAL, theta, theta_f16, mask,
                      results_dev, ws, kScratchBytes, stream, cfg, arena, true);
}

}  // extern "C" (reopened below)

namespace condensa {

static condensa_status lc_step_impl(bool pq, const condensa_tensor* tensors, int n_tensors, float* const* lambda,
                                    float* const* lambda_out, float mu, double density, float* const* theta,
                                    uint16_t* const* theta_f16, float* const* grad, uint8_t* const* mask,
                                    uint64_t* nnz_dev, condensa_select* result_dev, void* workspace_dev,
                                    size_t workspace_bytes, void* stream, const condensa_config* config) {
    Config cfg;
    condensa_status rc = resolve_config(config, &cfg);
    if (rc != CONDENSA_OK) return rc;
    if (result_dev == nullptr) return CONDENSA_ERR_NULL;
    if (n_tensors > 0 && lambda == nullptr) return CONDENSA_ERR_NULL;
    if (!density_ok(density)) return CONDENSA_ERR_DENSITY;
    if (!(mu > 0.0f) || !std::isfinite(mu)) return CONDENSA_ERR_DENSITY;
    HostArena arena;
    Tables tb;
    rc = build_tensor_table(tensors, n_tensors, &tb, arena);
    if (rc != CONDENSA_OK) return rc;
    Layout L = make_layout(CONDENSA_OP_LC_STEP, tb.N, 0, n_tensors, 1, CONDENSA_SCOPE_GLOBAL, cfg);

    std::vector<OutDesc> out(static_cast<size_t>(n_tensors > 0 ? n_tensors : 1), OutDesc{});
    std::vector<ByteRange> ranges;
    ranges.reserve(static_cast<size_t>(n_tensors) * 7 + 2);
    bool vec = tb.vec;
    bool in_place_any = false;
    for (int t = 0; t < n_tensors; ++t) {
        TensorDesc& d = tb.td[t];
        if (d.n == 0) continue;
        if (lambda[t] == nullptr) return CONDENSA_ERR_NULL;
        d.lam = lambda[t];
        d.lam_out = lambda_out ? lambda_out[t] : lambda[t];
        if (d.lam_out == nullptr) return CONDENSA_ERR_NULL;
        d.grad = grad ? grad[t] : nullptr;
        OutDesc& o = out[t];
        o.theta = theta ? theta[t] : nullptr;
        o.theta16 = (pq && theta_f16) ? theta_f16[t] : nullptr;
        o.mask = mask ? mask[t] : nullptr;
        // theta, grad, mask, theta16 and a separate lambda_out must be disjoint from everything else; lambda
        // updated in place is a written range, so it must not overlap the weights either
        const bool in_place = (d.lam_out == d.lam);
        in_place_any = in_place_any || in_place;
        ranges.push_back(byte_range(d.w, d.n * 4, false));
        ranges.push_back(byte_range(d.lam, d.n * 4, in_place));
        if (!in_place) ranges.push_back(byte_range(d.lam_out, d.n * 4, true));
        ranges.push_back(byte_range(o.theta, d.n * 4, true));
        ranges.push_back(byte_range(d.grad, d.n * 4, true));
        ranges.push_back(byte_range(o.mask, d.n, true));
        ranges.push_back(byte_range(o.theta16, d.n * 2, true));
        if (!aligned16(d.lam) || !aligned16(d.lam_out)) vec = false;
        if (o.theta && !aligned16(o.theta)) vec = false;
        if (d.grad && !aligned16(d.grad)) vec = false;
        if (o.mask && (reinterpret_cast<uintptr_t>(o.mask) & 3u)) vec = false;
        if (o.theta16 && (reinterpret_cast<uintptr_t>(o.theta16) & 7u)) vec = false;
    }
    if (in_place_any || cfg[CONDENSA_OPT_FUSED_SWEEP] != 0) prefer_window_for_two_sweeps(CONDENSA_OP_LC_STEP, tb.N, n_tensors, workspace_bytes, &cfg, &L);
    fewer_gathered_where_short(CONDENSA_OP_LC_STEP, tb.N, n_tensors, 1, CONDENSA_SCOPE_GLOBAL, workspace_bytes, cfg, &L);
    ranges.push_back(byte_range(workspace_dev, workspace_bytes < L.total ? workspace_bytes : L.total, true));
    ranges.push_back(byte_range(result_dev, sizeof(condensa_select), true));
    ranges.push_back(byte_range(nnz_dev, sizeof(uint64_t), true));
    if (ranges_conflict(ranges.data(), ranges.size())) return CONDENSA_ERR_ARG;
    rc = check_workspace(workspace_dev, workspace_bytes, L);
    if (rc != CONDENSA_OK) return rc;
    const bool window = want_window(tb.N, n_tensors, false, 1, cfg);
    Slot slot4[4];
    Slot& slot = slot4[0];
    init_slot(&slot, tb.N, kept_count(density, tb.N), window || L.listed ? 2u : 1u);
    if (window) init_sample_slots(slot4 + 1, slot, cfg[CONDENSA_OPT_WINDOW_MARGIN]);

    hipStream_t st = static_cast<hipStream_t>(stream);
    std::vector<char> lists;
    ListShape list_shape;
    const size_t list_bytes = L.listed ? build_list_table(tb, L, n_tensors, 1, false, true, cfg, &lists, &list_shape) : 0;
    // the selection sweeps read w and lambda only, so their vector path depends on those alone
    bool vec_in = tb.vec;
    for (int t = 0; t < n_tensors; ++t)
        if (tb.td[t].n > 0 && !aligned16(tb.td[t].lam)) vec_in = false;
    const OutDesc* od = at<OutDesc>(workspace_dev, L.out);
    const ListRequest rq{od, vec, pq, !in_place_any && cfg[CONDENSA_OPT_FUSED_SWEEP] == 0, pq ? nnz_dev : nullptr, false};
    bool sampled = false;
    StageImage img;
    if (L.listed)
        rc = vec_in ? begin_and_sample<true, true>(L, tb, n_tensors, out.data(), out.size(), slot4, &density, 1, false, mu, workspace_dev, st, lists, list_shape, rq, cfg, &img, &sampled)
                    : begin_and_sample<true, false>(L, tb, n_tensors, out.data(), out.size(), slot4, &density, 1, false, mu, workspace_dev, st, lists, list_shape, rq, cfg, &img, &sampled);
    if (rc == CONDENSA_OK && !sampled)
        rc = begin_call(L, tb, n_tensors, out.data(), out.size(), slot4, window ? 4 : 1, workspace_dev, st, &img, lists.data(), list_bytes);
    if (rc != CONDENSA_OK) return rc;

    DataArgs a{};
    a.td = at<TensorDesc>(workspace_dev, L.td);
    a.slots = at<Slot>(workspace_dev, L.slots);
    a.hist0 = at<u64>(workspace_dev, L.hist0);
    a.histx = at<u64>(workspace_dev, L.histx);
    a.coarse = at<u64>(workspace_dev, L.histc);
    a.tiecnt = at<u32>(workspace_dev, L.tiecnt);
    a.tiehit = at<u32>(workspace_dev, L.tiehit);
    if (L.tl_key) {
        a.tl_cnt = at<u64>(workspace_dev, L.tl_cnt);
        a.tl_key = at<u32>(workspace_dev, L.tl_key);
        a.tl_idx = at<u64>(workspace_dev, L.tl_idx);
    }
    a.ctl = at<Control>(workspace_dev, L.ctl);
    a.chunk_map = at<u32>(workspace_dev, L.chunk_map);
    a.n_chunks = tb.n_chunks;
    a.N = tb.N;
    a.n_tensors = n_tensors;
    a.J = 1;
    a.per_tensor = 0;
    a.only_failed = 0;
    a.streaming = (tb.N * 8u >= (static_cast<u64>(512) << 20)) ? 1 : 0;            // w and lambda: well beyond the 256 MB last-level cache
    a.mu = mu;
    a.merged = 1;
    // counters of the apply sweeps' non-zero codes: the last row of the segment counters (rows 1.. belong to the
    // sweeps of several densities, which the L-C step never runs)
    // (listed windows: the one row that their workspace holds)
    a.nnz_seg = (pq && nnz_dev) ? at<u64>(workspace_dev, L.seg) + (L.listed ? 0 : static_cast<size_t>(kSegs) * (1 + kMaxJ)) : nullptr;

    // Window path: selection and apply share one sweep unless lambda is updated in place (a failed window
    // needs the inputs again).
    const bool fuse = window && tb.n_chunks > 0 && slot.k > 0 && !in_place_any && cfg[CONDENSA_OPT_FUSED_SWEEP] == 0;
    WindowArgs wargs{};
    FusedRequest fr{od, vec, pq, &wargs};
    if (L.listed) {
        rc = vec_in ? launch_listed<true, true>(a, L, workspace_dev, list_shape, 1, 1, result_dev, rq, sampled, st, cfg)
                    : launch_listed<true, false>(a, L, workspace_dev, list_shape, 1, 1, result_dev, rq, sampled, st, cfg);
        if (rc != CONDENSA_OK || rq.write) return rc;
    } else
        rc = vec_in ? run_selection<true, true>(a, L, workspace_dev, window, 1, 1, result_dev, st, cfg, fuse ? &fr : nullptr)
                    : run_selection<true, false>(a, L, workspace_dev, window, 1, 1, result_dev, st, cfg, fuse ? &fr : nullptr);
    if (rc != CONDENSA_OK) return rc;

    if (fuse) {
        PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
        if (pq) hipLaunchKernelGGL((k_window_fixup<true, true>), dim3(wargs.n_segs * kFixupParts), dim3(kBlock), 0, st, a, wargs);
        else    hipLaunchKernelGGL((k_window_fixup<true, false>), dim3(wargs.n_segs * kFixupParts), dim3(kBlock), 0, st, a, wargs);
        CONDENSA_LAUNCH_CHECK();
        const u64 n_tiles = tb.n_chunks * (kChunk / 256);
        const dim3 grid(static_cast<unsigned>(n_tiles < 16384 ? n_tiles : 16384));
        if (pq && vec)  hipLaunchKernelGGL((k_lc_apply_gated<true, true>), grid, dim3(64), 0, st, a, od, n_tiles);
        else if (pq)    hipLaunchKernelGGL((k_lc_apply_gated<false, true>), grid, dim3(64), 0, st, a, od, n_tiles);
        else if (vec)   hipLaunchKernelGGL((k_lc_apply_gated<true, false>), grid, dim3(64), 0, st, a, od, n_tiles);
        else            hipLaunchKernelGGL((k_lc_apply_gated<false, false>), grid, dim3(64), 0, st, a, od, n_tiles);
        CONDENSA_LAUNCH_CHECK();
    } else if (tb.n_chunks > 0) {
        PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
        const int64_t at_opt = cfg[CONDENSA_OPT_APPLY_THREADS];
        const unsigned nc = static_cast<unsigned>(tb.n_chunks);
        // measured on the 1.2 G-weight workload: 64 threads 3.94 ms, 256 threads 4.28 ms, 128 threads 4.55 ms
        if (pq) {
            if (vec) hipLaunchKernelGGL((k_lc_apply<true, 64, true>), dim3(nc * (kChunk / 256)), dim3(64), 0, st, a, od);
            else     hipLaunchKernelGGL((k_lc_apply<false, 256, true>), dim3(nc * (kChunk / 1024)), dim3(256), 0, st, a, od);
        }
        else if (vec && at_opt == 256) hipLaunchKernelGGL((k_lc_apply<true, 256, false>), dim3(nc * (kChunk / 1024)), dim3(256), 0, st, a, od);
        else if (vec && at_opt == 128) hipLaunchKernelGGL((k_lc_apply<true, 128, false>), dim3(nc * (kChunk / 512)), dim3(128), 0, st, a, od);
        else if (vec)                  hipLaunchKernelGGL((k_lc_apply<true, 64, false>), dim3(nc * (kChunk / 256)), dim3(64), 0, st, a, od);
        else                           hipLaunchKernelGGL((k_lc_apply<false, 256, false>), dim3(nc * (kChunk / 1024)), dim3(256), 0, st, a, od);
        CONDENSA_LAUNCH_CHECK();
    }
    if (pq && nnz_dev) {
        hipLaunchKernelGGL(k_nnz_finish, dim3(1), dim3(kBlock), 0, st, a, at<u64>(workspace_dev, L.seg) + kSegs,
                           (fuse && tb.n_chunks > 0) ? 1 : 0, nnz_dev);
        CONDENSA_LAUNCH_CHECK();
    }
    return CONDENSA_OK;
}

}  // namespace condensa

extern "C" {

condensa_status condensa_lc_step(const condensa_tensor* tensors, int n_tensors, float* const* lambda,
                                 float* const* lambda_out, float mu, double density, float* const* theta,
                                 float* const* grad, uint8_t* const* mask, condensa_select* result_dev,
                                 void* workspace_dev, size_t workspace_bytes, void* stream,
                                 const condensa_config* config) {
    return lc_step_impl(false, tensors, n_tensors, lambda, lambda_out, mu, density, theta, nullptr, grad, mask,
                        nullptr, result_dev, workspace_dev, workspace_bytes, stream, config);
}

condensa_status condensa_lc_step_pq(const condensa_tensor* tensors, int n_tensors, float* const* lambda,
                                    float* const* lambda_out, float mu, double density, float* const* theta,
                                    uint16_t* const* theta_f16, float* const* grad, uint8_t* const* mask,
                                    uint64_t* nnz_dev, condensa_select* result_dev, void* workspace_dev,
                                    size_t workspace_bytes, void* stream, const condensa_config* config) {
    return lc_step_impl(true, tensors, n_tensors, lambda, lambda_out, mu, density, theta, theta_f16, grad, mask,
                        nnz_dev, result_dev, workspace_dev, workspace_bytes, stream, config);
}

condensa_status condensa_count_nonzero(const condensa_tensor* tensors, int n_tensors, int kind,
                                       uint64_t* count_dev, void* workspace_dev, size_t workspace_bytes,
                                       void* stream, const condensa_config* config) {
    Config cfg;
    condensa_status rc = resolve_config(config, &cfg);
    if (rc != CONDENSA_OK) return rc;
    if (count_dev == nullptr) return CONDENSA_ERR_NULL;
    if (kind < CONDENSA_COUNT_F32 || kind > CONDENSA_COUNT_CODES8) return CONDENSA_ERR_ARG;
    HostArena arena;
    Tables tb;
    rc = build_tensor_table(tensors, n_tensors, &tb, arena);
    if (rc != CONDENSA_OK) return rc;
    const Layout L = make_layout(CONDENSA_OP_COUNT_NONZERO, tb.N, 0, n_tensors, 1, CONDENSA_SCOPE_GLOBAL, cfg);
    rc = check_workspace(workspace_dev, workspace_bytes, L);
    if (rc != CONDENSA_OK) return rc;
    bool vec = true;
    std::vector<ByteRange> ranges;
    const u64 elem_bytes = kind == CONDENSA_COUNT_F32 ? 4 : (kind == CONDENSA_COUNT_CODES16 ? 2 : 1);
    for (int t = 0; t < n_tensors; ++t) {
        if (tb.td[t].n > 0 && (reinterpret_cast<uintptr_t>(tb.td[t].w) & 15u)) vec = false;
        ranges.push_back(byte_range(tb.td[t].w, tb.td[t].n * elem_bytes, false));
    }
    ranges.push_back(byte_range(workspace_dev, workspace_bytes < L.total ? workspace_bytes : L.total, true));
    ranges.push_back(byte_range(count_dev, sizeof(uint64_t), true));
    if (ranges_conflict(ranges.data(), ranges.size())) return CONDENSA_ERR_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    StageImage img;
    rc = begin_call(L, tb, n_tensors, nullptr, 0, nullptr, 0, workspace_dev, st, &img);
    if (rc != CONDENSA_OK) return rc;

    DataArgs a{};
    a.td = at<TensorDesc>(workspace_dev, L.td);
    a.chunk_map = at<u32>(workspace_dev, L.chunk_map);
    a.n_chunks = tb.n_chunks;
    a.N = tb.N;
    a.n_tensors = n_tensors;
    u64* partial = at<u64>(workspace_dev, L.hist0);            // kBins words, cleared by k_prepare
    const unsigned blocks = static_cast<unsigned>(tb.n_chunks < static_cast<u64>(kBins) ? (tb.n_chunks ? tb.n_chunks : 1) : kBins);
    if (tb.n_chunks > 0) {
        if (kind == CONDENSA_COUNT_CODES8) {
            if (vec) hipLaunchKernelGGL((k_count_nonzero<2, true>), dim3(blocks), dim3(kBlock), 0, st, a, partial);
            else     hipLaunchKernelGGL((k_count_nonzero<2, false>), dim3(blocks), dim3(kBlock), 0, st, a, partial);
        } else if (kind == CONDENSA_COUNT_CODES16) {
            if (vec) hipLaunchKernelGGL((k_count_nonzero<1, true>), dim3(blocks), dim3(kBlock), 0, st, a, partial);
            else     hipLaunchKernelGGL((k_count_nonzero<1, false>), dim3(blocks), dim3(kBlock), 0, st, a, partial);
        } else {
            if (vec) hipLaunchKernelGGL((k_count_nonzero<0, true>), dim3(blocks), dim3(kBlock), 0, st, a, partial);
            else     hipLaunchKernelGGL((k_count_nonzero<0, false>), dim3(blocks), dim3(kBlock), 0, st, a, partial);
        }
        CONDENSA_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, st, partial, blocks, count_dev);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}

}  // extern "C" (reopened below)

// ---- structure pruning (filters, 2-D blocks) ---------------------------------------------------------

namespace condensa {

// Lays the strips of every tensor when the call is one for them: GLOBAL scope (the layout has their regions), blocks of two dimensions and at most
// kStripArea elements, theta apart from the weights, a threshold strictly inside the population.  b2, b3: the widest blocks there are.  Larger blocks
// leave a strip's additions to a few threads (43 thousand of 32x32: 196 us, 130 with the aggregates first).  Every such call takes the strips: they are ahead
// from 4 thousand blocks (7 thousand of 5x5 31-36 -> 24 us; 45 thousand of 8x8, the threshold among the highest 2 %, 34-38 -> 32) to 2^24, but for thresholds at a gap
// (k_struct_strip.h: 2^20 blocks in two scales 74 -> 82 us), which no rule on sizes tells; beyond, and beyond 2^30 weights, nothing was measured and
// k_struct_fused.h or the radix levels go on.
struct StripPlan { u32 n_tiles = 0, b2 = 1, b3 = 1; bool quad = true; };
static bool strip_plan(Tables& tb, int n_tensors, const OutDesc* out, bool vec, const Slot& slot, const Layout& L, const Config& cfg, StripPlan* plan) {
    if (!L.strips || cfg[CONDENSA_OPT_FUSED_SWEEP] != 0 || n_tensors > static_cast<int>(kStripTensors) || slot.k == 0 || slot.k >= slot.n) return false;
    StripPlan p;
    p.quad = vec;
    bool any = false;
    for (int t = 0; t < n_tensors; ++t) {
        const TensorDesc& d = tb.td[t];
        if (d.n == 0) continue;
        if (d.d[0] != 1 || d.d[1] != 1 || d.b[0] != 1 || d.b[1] != 1 || d.d[3] > (1u << 26) || out[t].theta == d.w) return false;
        p.b2 = d.b[2] > p.b2 ? d.b[2] : p.b2;
        p.b3 = d.b[3] > p.b3 ? d.b[3] : p.b3;
        if (d.d[3] % 4 != 0 || d.b[3] % 4 != 0) p.quad = false;
        any = any || out[t].theta || out[t].mask;
    }
    if (!any || static_cast<u64>(p.b2) * p.b3 > kStripArea) return false;
    u64 tiles = 0;
    for (int t = 0; t < n_tensors; ++t) {
        TensorDesc& d = tb.td[t];
        if (d.n == 0) { d.reserved[0] = tiles; continue; }
        tiles += strip_layout(&d, p.quad, tiles);
    }
    if (tiles >= L.cand_cap) return false;                  // (their counts go where the list of blocks would)
    p.n_tiles = static_cast<u32>(tiles);
    *plan = p;
    return true;
}

static condensa_status run_strips(const Layout& L, const Tables& tb, int n_tensors, const std::vector<OutDesc>& out, const std::vector<Slot>& slots, const StripPlan& plan,
                                  double* sumsq_dev, float* norms_dev, int32_t* keep_idx_dev, uint8_t* structure_mask_dev, condensa_select* results_dev,
                                  void* ws, hipStream_t st, const Config& cfg) {
    const StripBins sb = strip_bins(tb.F);
    const u32 groups = strip_groups(tb.F), rounds = strip_rounds(tb.F, slots[0].k);
    const u32 log_group = plan.n_tiles < (1u << 14) ? 6u : 9u;           // a workgroup of k_strip_resolve adds up the counts of so many strips, and of all groups
    Layout Z = L;                                           // of the counters, only these are used
    Z.zero_begin = L.s_zero;
    Z.zero_bytes = L.s_coarse + align_up(((plan.n_tiles >> log_group) + 1) * kListLine * sizeof(u32)) - L.s_zero;
    StructArgs a{};
    a.td = at<TensorDesc>(ws, L.td);
    a.slots = at<Slot>(ws, L.slots);
    a.keys = at<u64>(ws, L.skeys);
    a.F = tb.F;
    a.n_tensors = n_tensors;
    ListArgs w{};
    w.local = at<u64>(ws, L.s_local);
    w.n_local = groups;
    w.tag = next_tag();
    w.win = at<ListWin>(ws, L.s_win);
    w.margin16 = static_cast<int>(cfg[CONDENSA_OPT_WINDOW_MARGIN]);
    w.force = t_force;
    StripArgs s{};
    s.win = w.win;
    s.hist = at<u32>(ws, L.s_hist);
    s.key = at<u64>(ws, L.s_key);
    s.id = at<u32>(ws, L.s_id);
    s.log_bins = sb.log_bins;
    s.log_room = sb.log_room;
    s.log_group = log_group;
    s.n_tiles = plan.n_tiles;
    s.above = at<u32>(ws, L.s_above);
    s.tiles = at<uint2>(ws, L.cand_idx);
    s.coarse = at<u32>(ws, L.s_coarse);
    s.pass = at<u32>(ws, L.s_pass);
    s.meet = at<u32>(ws, L.s_meet);
    s.share = at<u32>(ws, L.s_share);
    s.tie_end = reinterpret_cast<u64*>(s.share + 2 * kStripResolveGrid);
    s.out = at<OutDesc>(ws, L.out);
    s.keep_idx = keep_idx_dev;
    s.user_mask = structure_mask_dev;
    s.results = results_dev;
    s.quad = plan.quad ? 1 : 0;
    s.units = plan.b2 * plan.b3 / (plan.quad ? 4 : 1);
    s.by_units = make_fastdiv(s.units);
    StageImage img;
    const size_t td_bytes = static_cast<size_t>(tb.n_td) * sizeof(TensorDesc), out_bytes = out.size() * sizeof(OutDesc), slot_bytes = sizeof(Slot);
    const bool one = n_tensors <= kStripBeginTensors && td_bytes + out_bytes + slot_bytes <= kStageBytes;
    if (one) {
        const condensa_status rc = img.acquire(td_bytes + out_bytes + slot_bytes, st);
        if (rc != CONDENSA_OK) return rc;
    }
    if (one && img.data() != nullptr) {
        PhaseTimer timer(CONDENSA_PHASE_SAMPLE, st, cfg);
        StripBeginArgs b{};
        b.up = fill_image(img, Z, ws, tb, out.data(), out_bytes, slots.data(), slot_bytes, nullptr, 0);
        b.zero = at<uint4>(ws, Z.zero_begin);
        b.n_zero = Z.zero_bytes / 16;
        b.F = tb.F;
        b.k = slots[0].k;
        b.n_tensors = n_tensors;
        b.groups = groups;
        b.rounds = rounds;
        b.fillers = static_cast<u32>((b.n_zero + 2 * kStripBegin - 1) / (2 * kStripBegin));
        b.b2 = plan.b2;
        b.b3 = plan.b3;
        b.quad = s.quad;
        for (int t = 0; t < n_tensors; ++t) {
            b.w[t] = tb.td[t].w;
            b.d2[t] = tb.td[t].d[2];
            b.d3[t] = tb.td[t].d[3];
        }
        for (int t = 0; t <= n_tensors; ++t) b.start[t] = static_cast<u32>(tb.td[t].struct_start);
        img.launching(st);
        hipLaunchKernelGGL(k_strip_begin, dim3(1 + b.groups + b.fillers + 1), dim3(kStripBegin), 0, st, b, w);
        CONDENSA_LAUNCH_CHECK();
        img.commit();
    } else {
        const condensa_status rc = begin_call(Z, tb, n_tensors, out.data(), out.size(), slots.data(), 1, ws, st, &img);
        if (rc != CONDENSA_OK) return rc;
        PhaseTimer timer(CONDENSA_PHASE_SAMPLE, st, cfg);
        hipLaunchKernelGGL(k_strip_sample, dim3(groups), dim3(kStripBegin), 0, st, a, w, rounds, plan.b2, plan.b3, s.quad);
        CONDENSA_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_strip_bounds, dim3(1), dim3(64), 0, st, w, groups);
        CONDENSA_LAUNCH_CHECK();
    }
    {
        PhaseTimer timer(CONDENSA_PHASE_AGGREGATE, st, cfg);
        if (plan.quad) hipLaunchKernelGGL((k_struct_strips<true>), dim3(plan.n_tiles), dim3(kStripThreads), 0, st, a, s, sumsq_dev, norms_dev);
        else           hipLaunchKernelGGL((k_struct_strips<false>), dim3(plan.n_tiles), dim3(kStripThreads), 0, st, a, s, sumsq_dev, norms_dev);
        CONDENSA_LAUNCH_CHECK();
    }
    PhaseTimer timer(CONDENSA_PHASE_RESOLVE, st, cfg);
    u64 grid = (tb.F + kStripSettle - 1) / kStripSettle;
    if (grid > kStripResolveGrid) grid = kStripResolveGrid;
    for (int late = 0; late <= ((t_force & kForceLate) ? 1 : 0); ++late) {
        hipLaunchKernelGGL(k_strip_resolve, dim3(static_cast<unsigned>(grid)), dim3(kResolveThreads), 0, st, a, s);
        CONDENSA_LAUNCH_CHECK();
    }
    return CONDENSA_OK;
}

static condensa_status run_structure_prune(int op, Tables& tb, int n_tensors, double density, int scope,
                                           float* const* theta, uint8_t* const* mask, double* sumsq_dev,
                                           float* norms_dev, int32_t* keep_idx_dev, uint8_t* structure_mask_dev,
                                           condensa_select* results_dev, void* workspace_dev,
                                           size_t workspace_bytes, void* stream, const Config& cfg) {
    const bool per_tensor = (scope == CONDENSA_SCOPE_PER_TENSOR);
    if (per_tensor && n_tensors == 0) return CONDENSA_OK;
    Layout L = make_layout(op, tb.N, tb.F, n_tensors, 1, scope, cfg);
    // A workspace sized for another selection path, or for a population too large for strips, may lack their regions, which come last: the call goes without them.
    if (L.strips && workspace_bytes < L.total) {
        L.strips = false;
        L.total = L.s_zero;
    }

    std::vector<OutDesc> out(static_cast<size_t>(n_tensors > 0 ? n_tensors : 1), OutDesc{});
    std::vector<ByteRange> ranges;
    ranges.reserve(static_cast<size_t>(n_tensors) * 3 + 6);
    bool vec = tb.vec;
    for (int t = 0; t < n_tensors; ++t) {
        const u64 n = tb.td[t].n;
        if (n == 0) continue;
        OutDesc& o = out[t];
        o.theta = theta ? theta[t] : nullptr;
        o.mask = mask ? mask[t] : nullptr;
        const bool in_place = (o.theta == tb.td[t].w);       // the aggregates are complete before the apply sweep
        if (!in_place) ranges.push_back(byte_range(o.theta, n * 4, true));
        ranges.push_back(byte_range(o.mask, n, true));
        ranges.push_back(byte_range(tb.td[t].w, n * 4, in_place));
        if (o.theta && !aligned16(o.theta)) vec = false;
        if (o.mask && (reinterpret_cast<uintptr_t>(o.mask) & 3u)) vec = false;
    }
    ranges.push_back(byte_range(sumsq_dev, tb.F * 8, true));
    ranges.push_back(byte_range(norms_dev, tb.F * 4, true));
    ranges.push_back(byte_range(keep_idx_dev, tb.F * 4, true));
    ranges.push_back(byte_range(structure_mask_dev, tb.F, true));
    ranges.push_back(byte_range(workspace_dev, workspace_bytes < L.total ? workspace_bytes : L.total, true));
    ranges.push_back(byte_range(results_dev, static_cast<u64>(L.n_slots) * sizeof(condensa_select), true));
    if (ranges_conflict(ranges.data(), ranges.size())) return CONDENSA_ERR_ARG;
    condensa_status rc = check_workspace(workspace_dev, workspace_bytes, L);
    if (rc != CONDENSA_OK) return rc;
    std::vector<Slot> slots(static_cast<size_t>(L.n_slots) + 3);
    for (int g = 0; g < L.n_groups; ++g) {
        const u64 n = per_tensor ? tb.td[g].n_struct : tb.F;
        init_slot(&slots[g], n, kept_count(density, n), 1u);
    }
    StripPlan plan;
    if (strip_plan(tb, n_tensors, out.data(), vec, slots[0], L, cfg, &plan))
        return run_strips(L, tb, n_tensors, out, slots, plan, sumsq_dev, norms_dev, keep_idx_dev, structure_mask_dev, results_dev, workspace_dev,
                          static_cast<hipStream_t>(stream), cfg);
    // One sweep for aggregation AND apply (k_struct_fused.h): 8x8 blocks, every matrix a whole number of 64-block
    // runs wide, 128-bit accesses everywhere, outputs apart from the weights, a threshold strictly inside the
    // population, and enough blocks for the sample to pay (or the form asked for): 2^20 blocks take 218 us this way and
    // 181 with the aggregates first and a list (k_struct_list.h), 1.5 M blocks 262 and 258, 3.7 M blocks 487 and 606.  Strips
    // (above) come first: this is left with more than 2^24 blocks, 2^30 weights or 1024 tensors.
    bool fused = !per_tensor && (theta || mask) && vec && tb.F > kSmallGroup && slots[0].k > 0 && slots[0].k < tb.F &&
                 (cfg[CONDENSA_OPT_SELECT_PATH] == 2 || (cfg[CONDENSA_OPT_SELECT_PATH] == 0 && tb.F >= (static_cast<u64>(3) << 19))) &&
                 cfg[CONDENSA_OPT_FUSED_SWEEP] == 0;
    for (int t = 0; t < n_tensors && fused; ++t) {
        const TensorDesc& d = tb.td[t];
        if (d.n == 0) continue;
        const bool ok = d.d[0] == 1 && d.d[1] == 1 && d.b[2] == 8 && d.b[3] == 8 && d.d[2] % 8 == 0 && d.d[3] % 512 == 0 &&
                        aligned16(d.w) && d.n <= 0xFFFFFFFFull && out[t].theta != d.w;
        if (!ok) fused = false;
    }
    if (fused) {
        init_sample_slots(&slots[L.n_slots], slots[0], cfg[CONDENSA_OPT_WINDOW_MARGIN]);
        slots[0].path = 2;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    StructArgs a{};
    a.td = at<TensorDesc>(workspace_dev, L.td);
    a.slots = at<Slot>(workspace_dev, L.slots);
    a.histx = at<u64>(workspace_dev, L.histx);
    a.tiecnt = at<u32>(workspace_dev, L.tiecnt);
    a.ctl = at<Control>(workspace_dev, L.ctl);
    a.keys = at<u64>(workspace_dev, L.skeys);
    a.smask = at<u8>(workspace_dev, L.smask);
    a.sblock = at<u32>(workspace_dev, L.sblock);
    a.chunk_map = at<u32>(workspace_dev, L.chunk_map);
    a.F = tb.F;
    a.n_schunks = tb.n_schunks;
    a.n_chunks = tb.n_chunks;
    a.n_tensors = n_tensors;
    a.per_tensor = per_tensor ? 1 : 0;
    a.merged = per_tensor ? 0 : 1;
    a.hist_base = at<u64>(workspace_dev, L.hist0);
    a.coarse = at<u64>(workspace_dev, L.histc);

    // every structure one contiguous row (filters, neurons) of some length: staged, coalesced reads
    constexpr u64 kFewRowsMax = 32768;           // up to 1024 workgroups of kFewRows rows
    bool rows = tb.F > 0 && !fused && tb.N / tb.F >= 16;
    u64 loose = 0;                               // elements of tensors whose rows are not all 16-byte aligned
    u32 longest = 0;
    for (int t = 0; t < n_tensors && rows; ++t) {
        const TensorDesc& d = tb.td[t];
        if (d.n > 0 && d.d[3] > longest) longest = d.d[3];
        if (d.n > 0 && !(d.d[1] == 1 && d.d[2] == 1 && d.b[0] == 1 && d.b[3] == d.d[3])) rows = false;
        if (d.n > 0 && (d.d[3] % 4 != 0 || !aligned16(d.w))) loose += d.n;
    }
    StageImage img;
    const size_t n_slots_up = static_cast<size_t>(L.n_slots) + (fused ? 3 : 0);
    // Few tensors, few rows, none long: the aggregates are taken in the launch that begins the call, which saves some 3 us of 25 to 40.  More rows,
    // and every workgroup's look at the arguments, which lie in host memory, costs that again: 32 000 of 16 elements in 80 tensors take 50.0 us so
    // and 45.5 in two launches.  A row of 8 000 elements takes its workgroup 75 us alone, and the launch saved is hardly seen (64 of them: 102.5 us and
    // 102.8); 64 of 200 000 take 2 238 us so and 2 188 in two launches.
    bool begun = false;
    if (rows && tb.F <= kBeginRows && longest <= kBeginRowsLength && n_tensors <= kBeginRowsTensors) {
        const size_t td_bytes = static_cast<size_t>(tb.n_td) * sizeof(TensorDesc), out_bytes = out.size() * sizeof(OutDesc), slot_bytes = n_slots_up * sizeof(Slot);
        if (td_bytes + out_bytes + slot_bytes <= kStageBytes) {
            rc = img.acquire(td_bytes + out_bytes + slot_bytes, st);
            if (rc != CONDENSA_OK) return rc;
            begun = img.data() != nullptr;
        }
        if (begun) {
            PhaseTimer timer(CONDENSA_PHASE_AGGREGATE, st, cfg);
            BeginRowsArgs b{};
            b.begin = begin_tables_args(fill_image(img, L, workspace_dev, tb, out.data(), out_bytes, slots.data(), slot_bytes, nullptr, 0), L, tb, n_tensors, workspace_dev);
            const u64 fill = (b.begin.n_zero > tb.n_chunks ? b.begin.n_zero : tb.n_chunks) / (8 * kBlock) + 1;
            b.fillers = static_cast<u32>(fill < 256 ? fill : 256);
            for (int t = 0; t < n_tensors; ++t) {
                b.w[t] = tb.td[t].w;
                b.n[t] = tb.td[t].n;
                b.len[t] = tb.td[t].d[3];
                b.start[t] = static_cast<u32>(tb.td[t].struct_start);
                b.chunk_start[t] = static_cast<u32>(tb.td[t].chunk_start);
            }
            b.chunk_start[n_tensors] = static_cast<u32>(tb.n_chunks);
            const dim3 grid(static_cast<unsigned>(1 + b.fillers + (tb.F + kFewRows - 1) / kFewRows));
            img.launching(st);
            hipLaunchKernelGGL(k_begin_rows, grid, dim3(kBlock), 0, st, b, a, sumsq_dev, norms_dev);
            CONDENSA_LAUNCH_CHECK();
            img.commit();
        }
    }
    if (!begun) {
        rc = begin_call(L, tb, n_tensors, out.data(), out.size(), slots.data(), n_slots_up, workspace_dev, st, &img);
        if (rc != CONDENSA_OK) return rc;
    }
    const unsigned sblocks = static_cast<unsigned>((tb.F + kBlock - 1) / kBlock);
    const unsigned mtiles = static_cast<unsigned>((tb.F + kMaskTile - 1) / kMaskTile);
    // groups of at most kSmallGroup structures: one workgroup per group ranks, masks and lists them
    bool small = tb.F > 0 && cfg[CONDENSA_OPT_SELECT_PATH] != 1;
    if (per_tensor) { for (int t = 0; t < n_tensors && small; ++t) if (tb.td[t].n_struct > kSmallGroup) small = false; }
    else if (tb.F > kSmallGroup) small = false;
    bool finished = false;                                  // the ranking's record is written (k_struct_list_finish)
    StructWindowArgs sw{};
    if (fused) {
        sw.sample = at<u32>(workspace_dev, L.sample);
        sw.n_units = (L.sample_cap < tb.F ? L.sample_cap : tb.F) & ~static_cast<u64>(3);   // whole units of four blocks
        sw.stride = tb.F / sw.n_units;
        sw.wslots = a.slots + L.n_slots;
        sw.seg_cnt = at<u64>(workspace_dev, L.seg);
        sw.seg_above = sw.seg_cnt + kSegs;
        sw.cand_id = at<u32>(workspace_dev, L.cand_key);
        sw.cand_key = at<u64>(workspace_dev, L.cand_idx);
        sw.n_segs = sblocks < static_cast<unsigned>(kSegs) ? sblocks : static_cast<unsigned>(kSegs);   // at most the sweep's grid
        sw.seg_cap = L.cand_cap / sw.n_segs;
        sw.out = at<OutDesc>(workspace_dev, L.out);
        PhaseTimer timer(CONDENSA_PHASE_SAMPLE, st, cfg);
        ArrayArgs ar{};
        ar.keys = sw.sample; ar.n_host = sw.n_units; ar.slots = sw.wslots; ar.n_slots = 3;
        ar.hist = a.histx + static_cast<u64>(kStructLevels) * kBins;          // [2][3], behind the aggregate ranking's histograms
        ar.shared0 = ar.hist + static_cast<u64>(6) * kBins;
        ar.key_bits = 31; ar.merged = 1;
        ar.hist_base = at<u64>(workspace_dev, L.hist0); ar.coarse = at<u64>(workspace_dev, L.histc);
        u64 sg = (sw.n_units + kSampleHistThreads - 1) / kSampleHistThreads;
        if (sg > 512) sg = 512;
        hipLaunchKernelGGL(k_struct_sample_hist, dim3(static_cast<unsigned>(sg)), dim3(kSampleHistThreads), 0, st, a, sw, ar);
        CONDENSA_LAUNCH_CHECK();
        hipLaunchKernelGGL((k_hist_array<false>), dim3(hist_array_grid(ar.n_host)), dim3(kArrayThreads), 0, st, ar, 1);
        CONDENSA_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_window_bounds, dim3(1), dim3(kBlock), 0, st, ar);
        CONDENSA_LAUNCH_CHECK();
    }
    if (tb.F > 0) {
        if (!begun) {
            PhaseTimer timer(CONDENSA_PHASE_AGGREGATE, st, cfg);
            // Not all of them aligned, 256 rows to a workgroup or 64.  256: rows of one piece (a million of 17 elements 132 us the call, 149
            // with 64; of 33, 140 and 175; 40 thousand 39 and 37), and few loose ones among short ones of which there are very many (a
            // million of 256 and 40 of 33: 604 and 618) or among short and long ones where no compute unit gets a workgroup more than the
            // others (65 536 of 4608 and 40 of 33: 645 and 674; 100 thousand of 512: 192 and 137; 262 144 of 1024: 644 and 605).
            const u64 by_256 = (tb.F + 255) / 256 % 256, len = tb.N / tb.F;
            const bool even = by_256 <= 8 || by_256 >= 248;
            const bool mixed_by_256 = (len <= 33 && tb.F >= (1u << 16)) ||
                                      (loose <= tb.N / 12 && ((len <= 256 && (even || tb.F >= (1u << 19))) || (len >= 4096 && even)));
            // every tensor a matrix tiled exactly by 2-D blocks of one width of 4, 8, 16 or 32, rows 16-byte aligned
            u32 tile_w = 0;
            bool tiles = !rows;
            for (int t = 0; t < n_tensors && tiles; ++t) {
                const TensorDesc& d = tb.td[t];
                if (d.n == 0) continue;
                const bool ok = d.d[0] == 1 && d.d[1] == 1 && d.d[2] % d.b[2] == 0 && d.d[3] % d.b[3] == 0 &&
                                (d.b[3] == 4 || d.b[3] == 8 || d.b[3] == 16 || d.b[3] == 32) && (tile_w == 0 || tile_w == d.b[3]) &&
                                aligned16(d.w) && d.d[3] % 4 == 0 && d.n <= 0xFFFFFFFFull;
                if (!ok) tiles = false;
                tile_w = d.b[3];
            }
            if (fused && cfg[CONDENSA_OPT_APPLY_THREADS] == 256)
                hipLaunchKernelGGL((k_struct_tiles_fused<256>), dim3(sblocks), dim3(256), 0, st, a, sw, sumsq_dev, norms_dev);
            else if (fused && cfg[CONDENSA_OPT_APPLY_THREADS] == 128)
                hipLaunchKernelGGL((k_struct_tiles_fused<128>), dim3(static_cast<unsigned>((tb.F + 127) / 128)), dim3(128), 0, st, a, sw, sumsq_dev, norms_dev);
            else if (fused)
                hipLaunchKernelGGL((k_struct_tiles_fused<64>), dim3(static_cast<unsigned>((tb.F + 63) / 64)), dim3(64), 0, st, a, sw, sumsq_dev, norms_dev);
            else if (rows && tb.F <= 512 * kFewRows)
                hipLaunchKernelGGL((k_struct_sumsq_rows_few<true, kFewRows>), dim3(static_cast<unsigned>((tb.F + kFewRows - 1) / kFewRows)), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (rows && tb.F <= kFewRowsMax)
                hipLaunchKernelGGL((k_struct_sumsq_rows_few<false, kFewRows>), dim3(static_cast<unsigned>((tb.F + kFewRows - 1) / kFewRows)), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (rows && loose == 0) hipLaunchKernelGGL(k_struct_sumsq_rows<false>, dim3(sblocks), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (rows && mixed_by_256) hipLaunchKernelGGL(k_struct_sumsq_rows<true>, dim3(sblocks), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (rows) hipLaunchKernelGGL((k_struct_sumsq_rows_few<false, kManyRows>), dim3(static_cast<unsigned>((tb.F + kManyRows - 1) / kManyRows)), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (tiles && tile_w == 4)  hipLaunchKernelGGL((k_struct_sumsq_tiles<1>), dim3(sblocks), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (tiles && tile_w == 8)  hipLaunchKernelGGL((k_struct_sumsq_tiles<2>), dim3(sblocks), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (tiles && tile_w == 16) hipLaunchKernelGGL((k_struct_sumsq_tiles<4>), dim3(sblocks), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else if (tiles && tile_w == 32) hipLaunchKernelGGL((k_struct_sumsq_tiles<8>), dim3(sblocks), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            else      hipLaunchKernelGGL(k_struct_sumsq, dim3(sblocks), dim3(kBlock), 0, st, a, sumsq_dev, norms_dev);
            CONDENSA_LAUNCH_CHECK();
        }
        PhaseTimer timer(CONDENSA_PHASE_RESOLVE, st, cfg);
        if (small) {
            hipLaunchKernelGGL(k_struct_small, dim3(L.n_slots), dim3(kSmallThreads), 0, st, a, structure_mask_dev,
                               keep_idx_dev, results_dev);
            CONDENSA_LAUNCH_CHECK();
        }
        if (fused) {
            // rank k - (blocks above the window) among the listed blocks; the levels over all aggregates below are
            // then the fallback and return at once
            hipLaunchKernelGGL(k_struct_window_check, dim3(1), dim3(kBlock), 0, st, a, sw);
            CONDENSA_LAUNCH_CHECK();
            const unsigned lg = sw.n_segs < 256 ? sw.n_segs : 256;
            for (int level = 0; level < n_levels(63); ++level) {
                hipLaunchKernelGGL(k_hist_listed_keys, dim3(lg), dim3(kArrayThreads), 0, st, a, sw, level);
                CONDENSA_LAUNCH_CHECK();
            }
            a.only_failed = 1;
        }
        // moderate rankings on the automatic path: one histogram over all aggregates, then a list (k_struct_list.h)
        const bool listed = !per_tensor && !small && !fused && tb.F <= kSmallCallElems && cfg[CONDENSA_OPT_SELECT_PATH] == 0;
        const u64 pieces = a.merged ? (tb.F + kKeyPiece - 1) / kKeyPiece : tb.n_schunks;
        u64 cpb = (pieces + 1023) / 1024;
        if (a.merged && cpb < 4) cpb = 4;                    // fewer workgroups, fewer of them adding to the same 2048 counters
        const u64 blocks = (pieces + cpb - 1) / (cpb ? cpb : 1);
        for (int level = 0; level < n_levels(63) && !small && !listed; ++level) {
            hipLaunchKernelGGL(k_hist_keys, dim3(static_cast<unsigned>(blocks)), dim3(kBlock), 0, st, a, level, cpb);
            CONDENSA_LAUNCH_CHECK();
            if (a.merged) continue;                            // the next kernel folds this level in itself
            hipLaunchKernelGGL(k_scan_level, dim3(L.n_slots), dim3(kBlock), 0, st, a.slots,
                               static_cast<const u64*>(nullptr), a.histx, 1, 63, level, a.ctl, 0, &a.ctl->need_tie);
            CONDENSA_LAUNCH_CHECK();
        }
        if (listed) {
            StructListArgs l{};
            l.count = at<u64>(workspace_dev, L.seg);
            l.key = at<u64>(workspace_dev, L.cand_idx);
            l.id = at<u32>(workspace_dev, L.cand_key);
            l.cap = L.cand_cap;
            l.window = reinterpret_cast<u32*>(l.count + 1);
            l.piece = at<StructPiece>(workspace_dev, L.sample);          // (the sample of the one-sweep form, unused here)
            static_assert(kMaxPieces * sizeof(StructPiece) <= (kSmallCallElems / 8) * sizeof(u32) && 2 * sizeof(StructPiece) <= (sizeof(u32) << 12),
                          "a piece for every kKeyPiece structures fits a sample of an eighth of them, 4096 at least");
            // each workgroup adds most of 2048 bins to the ranking's histogram (688 128 keys of one radix level: 336 workgroups
            // took 16.4 us, 120 of them 10.7)
            u64 hb = pieces < 96 ? pieces : 96;
            const u64 ppb = (pieces + hb - 1) / hb;
            hb = (pieces + ppb - 1) / ppb;
            hipLaunchKernelGGL(k_struct_list_hist, dim3(static_cast<unsigned>(hb)), dim3(kBlock), 0, st, a, l, ppb);
            CONDENSA_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_struct_list_collect, dim3(static_cast<unsigned>(pieces < 1024 ? pieces : 1024)), dim3(kBlock), 0, st, a, l);
            CONDENSA_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_struct_list_finish, dim3(1), dim3(kSmallFinishThreads), 0, st, a, l, results_dev, bits_for(tb.F - 1));
            CONDENSA_LAUNCH_CHECK();
            finished = true;
        } else if (!small) {
            hipLaunchKernelGGL(k_tie_count_keys, dim3(static_cast<unsigned>(tb.n_schunks)), dim3(kBlock), 0, st, a);
            CONDENSA_LAUNCH_CHECK();
        }
    }
    if (!small && !finished) {
        hipLaunchKernelGGL(k_tie_locate_keys, dim3(L.n_slots), dim3(kBlock), 0, st, a, results_dev);
        CONDENSA_LAUNCH_CHECK();
    }
    if (tb.F > 0) {
        if (fused) {
            // the sweep left the keep flags of the blocks outside the window, the fix-up settles the listed ones
            // (and rewrites their theta and mask); the flags come from the keys only if the window failed
            PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
            hipLaunchKernelGGL(k_struct_fixup, dim3(sw.n_segs * kFixupParts), dim3(kBlock), 0, st, a, sw);
            CONDENSA_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_struct_mask, dim3(mtiles), dim3(kBlock), 0, st, a, structure_mask_dev, static_cast<int>(kMaskFromFlags));
            CONDENSA_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_struct_mask, dim3(mtiles), dim3(kBlock), 0, st, a, structure_mask_dev, static_cast<int>(kMaskIfFailed));
            CONDENSA_LAUNCH_CHECK();
        } else if (!small) {
            hipLaunchKernelGGL(k_struct_mask, dim3(mtiles), dim3(kBlock), 0, st, a, structure_mask_dev, static_cast<int>(kMaskFromKeys));
            CONDENSA_LAUNCH_CHECK();
        }
        const bool scanned = mtiles > kIdTilesDirect, apply = !fused && (theta || mask) && tb.n_chunks > 0;
        const u32 id_tiles = keep_idx_dev && !small ? mtiles : 0;
        if (id_tiles && scanned) {
            hipLaunchKernelGGL(k_struct_scan_blocks, dim3(1), dim3(kScanThreads), 0, st, a.sblock, static_cast<u64>(mtiles));
            CONDENSA_LAUNCH_CHECK();
        }
        if (id_tiles && !apply) {                           // otherwise in the apply sweep's launch
            hipLaunchKernelGGL(k_struct_keep_idx, dim3(id_tiles), dim3(kBlock), 0, st, a, keep_idx_dev, scanned ? 1 : 0);
            CONDENSA_LAUNCH_CHECK();
        }
        if (fused) {
            PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
            const OutDesc* od = at<OutDesc>(workspace_dev, L.out);
            const u64 n_tiles = tb.n_chunks * kSubPerChunk;
            hipLaunchKernelGGL((k_struct_apply_gated<true>), dim3(static_cast<unsigned>(n_tiles < 4096 ? n_tiles : 4096)), dim3(kBlock), 0, st, a, od, n_tiles);
            CONDENSA_LAUNCH_CHECK();
        } else if (apply) {
            PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
            const OutDesc* od = at<OutDesc>(workspace_dev, L.out);
            const dim3 grid(static_cast<unsigned>(tb.n_chunks * kSubPerChunk + id_tiles));
            if (vec) hipLaunchKernelGGL((k_struct_apply<true>), grid, dim3(kBlock), 0, st, a, od, keep_idx_dev, id_tiles, scanned ? 1 : 0);
            else     hipLaunchKernelGGL((k_struct_apply<false>), grid, dim3(kBlock), 0, st, a, od, keep_idx_dev, id_tiles, scanned ? 1 : 0);
            CONDENSA_LAUNCH_CHECK();
        }
    }
    return CONDENSA_OK;
}

enum StructKind { kFilters, kNeurons, kNeuronsAndFilters, kBlocks2D, kBlocksND };

// Fills the structure geometry of the tensor table.  Every tensor is seen as 4-D (leading dims 1)
// with a 4-D block; a filter / neuron is the block [1,1,1,len] of the tensor viewed as [F,1,1,len].
static condensa_status add_structure_geometry(const condensa_tensor* tensors, int n_tensors, StructKind kind,
                                              const int32_t* block, int block_ndim, Tables* tb) {
    u64 F = 0, sc = 0;
    for (int t = 0; t < n_tensors; ++t) {
        TensorDesc& d = tb->td[t];
        const condensa_tensor& T = tensors[t];
        d.struct_start = F;
        d.pad = sc;
        for (int i = 0; i < 4; ++i) { d.d[i] = 1; d.b[i] = 1; }
        u64 f = 0;
        if (kind == kFilters || kind == kNeurons || kind == kNeuronsAndFilters) {
            const bool ok = (kind == kFilters) ? T.ndim == 4 : (kind == kNeurons) ? T.ndim == 2 : (T.ndim == 2 || T.ndim == 4);
            if (!ok) return CONDENSA_ERR_SHAPE;
            if (d.n > 0) {
                f = static_cast<u64>(T.shape[0]);
                const u64 len = d.n / f;
                if (len > 0x7FFFFFFFull || f > 0x7FFFFFFFull) return CONDENSA_ERR_SIZE;
                d.d[0] = static_cast<u32>(f); d.d[3] = static_cast<u32>(len); d.b[3] = static_cast<u32>(len);
            }
        } else {
            if (T.ndim != block_ndim) return CONDENSA_ERR_SHAPE;
            const int pad = 4 - T.ndim;
            f = d.n > 0 ? 1 : 0;
            for (int i = 0; i < T.ndim; ++i) {
                const u64 dim = static_cast<u64>(T.shape[i]), blk = static_cast<u64>(block[i]);
                if (dim > 0x7FFFFFFFull) return CONDENSA_ERR_SIZE;
                if (kind == kBlocks2D && dim % blk != 0) return CONDENSA_ERR_SHAPE;
                if (d.n > 0) {
                    d.d[pad + i] = static_cast<u32>(dim);
                    d.b[pad + i] = static_cast<u32>(blk < dim ? blk : dim);
                    f *= (dim + blk - 1) / blk;
                }
            }
        }
        d.fd[kDivD1] = make_fastdiv(d.d[1]); d.fd[kDivD2] = make_fastdiv(d.d[2]); d.fd[kDivD3] = make_fastdiv(d.d[3]);
        d.fd[kDivB0] = make_fastdiv(d.b[0]); d.fd[kDivB1] = make_fastdiv(d.b[1]);
        d.fd[kDivB2] = make_fastdiv(d.b[2]); d.fd[kDivB3] = make_fastdiv(d.b[3]);
        d.n_struct = f;
        F += f;
        sc += (f + kChunk - 1) / kChunk;
    }
    if (F > 0x7FFFFFFFull) return CONDENSA_ERR_SIZE;         // ids are reported as int32
    tb->td[n_tensors].struct_start = F;
    tb->td[n_tensors].pad = sc;
    tb->F = F;
    tb->n_schunks = sc;
    return CONDENSA_OK;
}

static condensa_status structure_entry(StructKind kind, int op, const condensa_tensor* tensors, int n_tensors,
                                       const int32_t* block, int block_ndim, double density, int scope,
                                       float* const* theta, uint8_t* const* mask, double* sumsq_dev,
                                       float* norms_dev, int32_t* keep_idx_dev, uint8_t* structure_mask_dev,
                                       condensa_select* results_dev, void* workspace_dev, size_t workspace_bytes,
                                       void* stream, const condensa_config* config) {
    Config cfg;
    condensa_status rc = resolve_config(config, &cfg);
    if (rc != CONDENSA_OK) return rc;
    if (results_dev == nullptr) return CONDENSA_ERR_NULL;
    if (scope != CONDENSA_SCOPE_GLOBAL && scope != CONDENSA_SCOPE_PER_TENSOR) return CONDENSA_ERR_ARG;
    if (!density_ok(density)) return CONDENSA_ERR_DENSITY;
    if (kind == kBlocks2D || kind == kBlocksND) {
        if (block == nullptr) return CONDENSA_ERR_NULL;
        if (block_ndim < 1 || block_ndim > 4) return CONDENSA_ERR_SHAPE;
        for (int i = 0; i < block_ndim; ++i)
            if (block[i] < 1) return CONDENSA_ERR_SHAPE;
    }
    HostArena arena;
    Tables tb;
    rc = build_tensor_table(tensors, n_tensors, &tb, arena);
    if (rc != CONDENSA_OK) return rc;
    rc = add_structure_geometry(tensors, n_tensors, kind, block, block_ndim, &tb);
    if (rc != CONDENSA_OK) return rc;
    return run_structure_prune(op, tb, n_tensors, density, scope, theta, mask, sumsq_dev, norms_dev, keep_idx_dev,
                               structure_mask_dev, results_dev, workspace_dev, workspace_bytes, stream, cfg);
}

}  // namespace condensa

extern "C" {

condensa_status condensa_filter_prune(const condensa_tensor* tensors, int n_tensors, double density, int scope,
                                      float* const* theta, uint8_t* const* mask, double* sumsq_dev,
                                      float* norms_dev, int32_t* keep_idx_dev, uint8_t* structure_mask_dev,
                                      condensa_select* results_dev, void* workspace_dev, size_t workspace_bytes,
                                      void* stream,
                                      const condensa_config* config) {
    return structure_entry(kFilters, CONDENSA_OP_FILTER_PRUNE, tensors, n_tensors, nullptr, 0, density, scope, theta,
                           mask, sumsq_dev, norms_dev, keep_idx_dev, structure_mask_dev, results_dev, workspace_dev,
                           workspace_bytes, stream, config);
}

condensa_status condensa_neuron_prune(const condensa_tensor* tensors, int n_tensors, double density, int scope,
                                      float* const* theta, uint8_t* const* mask, double* sumsq_dev,
                                      float* norms_dev, int32_t* keep_idx_dev, uint8_t* structure_mask_dev,
                                      condensa_select* results_dev, void* workspace_dev, size_t workspace_bytes,
                                      void* stream,
                                      const condensa_config* config) {
    return structure_entry(kNeurons, CONDENSA_OP_FILTER_PRUNE, tensors, n_tensors, nullptr, 0, density, scope, theta,
                           mask, sumsq_dev, norms_dev, keep_idx_dev, structure_mask_dev, results_dev, workspace_dev,
                           workspace_bytes, stream, config);
}

condensa_status condensa_structure_prune(const condensa_tensor* tensors, int n_tensors, double density, int scope,
                                         float* const* theta, uint8_t* const* mask, double* sumsq_dev,
                                         float* norms_dev, int32_t* keep_idx_dev, uint8_t* structure_mask_dev,
                                         condensa_select* results_dev, void* workspace_dev, size_t workspace_bytes,
                                         void* stream,
                                      const condensa_config* config) {
    return structure_entry(kNeuronsAndFilters, CONDENSA_OP_FILTER_PRUNE, tensors, n_tensors, nullptr, 0, density, scope,
                           theta, mask, sumsq_dev, norms_dev, keep_idx_dev, structure_mask_dev, results_dev,
                           workspace_dev, workspace_bytes, stream, config);
}

condensa_status condensa_block_prune(const condensa_tensor* tensors, int n_tensors, int block_h, int block_w,
                                     double density, int scope, float* const* theta, uint8_t* const* mask,
                                     double* sumsq_dev, float* norms_dev, int32_t* keep_idx_dev,
                                     uint8_t* structure_mask_dev, condensa_select* results_dev,
                                     void* workspace_dev, size_t workspace_bytes, void* stream,
                                      const condensa_config* config) {
    const int32_t block[2] = {block_h, block_w};
    return structure_entry(kBlocks2D, CONDENSA_OP_BLOCK_PRUNE, tensors, n_tensors, block, 2, density, scope, theta,
                           mask, sumsq_dev, norms_dev, keep_idx_dev, structure_mask_dev, results_dev, workspace_dev,
                           workspace_bytes, stream, config);
}

condensa_status condensa_block_prune_nd(const condensa_tensor* tensors, int n_tensors, const int32_t* block_shape,
                                        int block_ndim, double density, int scope, float* const* theta,
                                        uint8_t* const* mask, double* sumsq_dev, float* norms_dev,
                                        int32_t* keep_idx_dev, uint8_t* structure_mask_dev,
                                        condensa_select* results_dev, void* workspace_dev, size_t workspace_bytes,
                                        void* stream,
                                      const condensa_config* config) {
    return structure_entry(kBlocksND, CONDENSA_OP_BLOCK_PRUNE, tensors, n_tensors, block_shape, block_ndim, density,
                           scope, theta, mask, sumsq_dev, norms_dev, keep_idx_dev, structure_mask_dev, results_dev,
                           workspace_dev, workspace_bytes, stream, config);
}

}  // extern "C"

namespace condensa {
template <typename C>
static condensa_status quantize_impl(const float* x_dev, uint64_t n, uint16_t* q_dev, float* dq_dev, void* stream) {
    if (n > kMaxElems) return CONDENSA_ERR_SIZE;
    if (n == 0) return CONDENSA_OK;
    if (q_dev == nullptr && dq_dev == nullptr) return CONDENSA_ERR_NULL;
    if (x_dev == nullptr) return CONDENSA_ERR_NULL;
    const bool vec = aligned16(x_dev) && (!dq_dev || aligned16(dq_dev)) &&
                     (!q_dev || (reinterpret_cast<uintptr_t>(q_dev) & 7u) == 0);
    constexpr int QT = kQuantThreads;
    const u64 blocks = (n + QT * 4 - 1) / (QT * 4);           // x QT threads stays below 2^32 for n <= kMaxElems
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!dq_dev && aligned16(x_dev) && aligned16(q_dev))
        hipLaunchKernelGGL((k_quantize_codes<QT, C>), dim3(static_cast<unsigned>((n + QT * 8 - 1) / (QT * 8))), dim3(QT), 0, st, x_dev, n, q_dev);
    else if (vec) hipLaunchKernelGGL((k_quantize<true, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, x_dev, n, q_dev, dq_dev);
    else     hipLaunchKernelGGL((k_quantize<false, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, x_dev, n, q_dev, dq_dev);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}

template <typename C>
static condensa_status dequantize_impl(const uint16_t* q_dev, uint64_t n, float* dq_dev, void* stream) {
    if (n > kMaxElems) return CONDENSA_ERR_SIZE;
    if (n == 0) return CONDENSA_OK;
    if (dq_dev == nullptr || q_dev == nullptr) return CONDENSA_ERR_NULL;
    const bool vec = aligned16(dq_dev) && (reinterpret_cast<uintptr_t>(q_dev) & 7u) == 0;
    constexpr int QT = kQuantThreads;
    const u64 blocks = (n + QT * 4 - 1) / (QT * 4);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (aligned16(q_dev) && aligned16(dq_dev))
        hipLaunchKernelGGL((k_dequantize_wide<QT, C>), dim3(static_cast<unsigned>((n + QT * 8 - 1) / (QT * 8))), dim3(QT), 0, st, q_dev, n, dq_dev);
    else if (vec) hipLaunchKernelGGL((k_dequantize<true, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, q_dev, n, dq_dev);
    else     hipLaunchKernelGGL((k_dequantize<false, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, q_dev, n, dq_dev);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}
template <typename C>
static condensa_status quantize8_impl(const float* x_dev, uint64_t n, uint8_t* q_dev, float* dq_dev, void* stream) {
    if (n > kMaxElems) return CONDENSA_ERR_SIZE;
    if (n == 0) return CONDENSA_OK;
    if (q_dev == nullptr && dq_dev == nullptr) return CONDENSA_ERR_NULL;
    if (x_dev == nullptr) return CONDENSA_ERR_NULL;
    const bool vec = aligned16(x_dev) && (!dq_dev || aligned16(dq_dev)) &&
                     (!q_dev || (reinterpret_cast<uintptr_t>(q_dev) & 3u) == 0);
    constexpr int QT = kQuantThreads;
    const u64 blocks = (n + QT * 4 - 1) / (QT * 4);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!dq_dev && aligned16(x_dev) && aligned16(q_dev))
        hipLaunchKernelGGL((k_quantize8_codes<QT, C>), dim3(static_cast<unsigned>((n + QT * 16 - 1) / (QT * 16))), dim3(QT), 0, st, x_dev, n, q_dev);
    else if (vec) hipLaunchKernelGGL((k_quantize8<true, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, x_dev, n, q_dev, dq_dev);
    else     hipLaunchKernelGGL((k_quantize8<false, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, x_dev, n, q_dev, dq_dev);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}

template <typename C>
static condensa_status dequantize8_impl(const uint8_t* q_dev, uint64_t n, float* dq_dev, void* stream) {
    if (n > kMaxElems) return CONDENSA_ERR_SIZE;
    if (n == 0) return CONDENSA_OK;
    if (dq_dev == nullptr || q_dev == nullptr) return CONDENSA_ERR_NULL;
    const bool vec = aligned16(dq_dev) && (reinterpret_cast<uintptr_t>(q_dev) & 3u) == 0;
    constexpr int QT = kQuantThreads;
    const u64 blocks = (n + QT * 4 - 1) / (QT * 4);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (aligned16(q_dev) && aligned16(dq_dev))
        hipLaunchKernelGGL((k_dequantize8_wide<QT, C>), dim3(static_cast<unsigned>((n + QT * 16 - 1) / (QT * 16))), dim3(QT), 0, st, q_dev, n, dq_dev);
    else if (vec) hipLaunchKernelGGL((k_dequantize8<true, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, q_dev, n, dq_dev);
    else     hipLaunchKernelGGL((k_dequantize8<false, QT, C>), dim3(static_cast<unsigned>(blocks)), dim3(QT), 0, st, q_dev, n, dq_dev);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}
}  // namespace condensa

extern "C" {

condensa_status condensa_quantize_fp8(const float* x_dev, uint64_t n, int format, uint8_t* q_dev, float* dq_dev,
                                      void* stream) {
    if (format == CONDENSA_FP8_E4M3) return quantize8_impl<CodecE4M3>(x_dev, n, q_dev, dq_dev, stream);
    if (format == CONDENSA_FP8_E5M2) return quantize8_impl<CodecE5M2>(x_dev, n, q_dev, dq_dev, stream);
    return CONDENSA_ERR_ARG;
}

condensa_status condensa_dequantize_fp8(const uint8_t* q_dev, uint64_t n, int format, float* dq_dev, void* stream) {
    if (format == CONDENSA_FP8_E4M3) return dequantize8_impl<CodecE4M3>(q_dev, n, dq_dev, stream);
    if (format == CONDENSA_FP8_E5M2) return dequantize8_impl<CodecE5M2>(q_dev, n, dq_dev, stream);
    return CONDENSA_ERR_ARG;
}

condensa_status condensa_quantize(const float* x_dev, uint64_t n, uint16_t* q_dev, float* dq_dev, void* stream) {
    return quantize_impl<CodecF16>(x_dev, n, q_dev, dq_dev, stream);
}

condensa_status condensa_dequantize(const uint16_t* q_dev, uint64_t n, float* dq_dev, void* stream) {
    return dequantize_impl<CodecF16>(q_dev, n, dq_dev, stream);
}

condensa_status condensa_quantize_bf16(const float* x_dev, uint64_t n, uint16_t* q_dev, float* dq_dev, void* stream) {
    return quantize_impl<CodecBF16>(x_dev, n, q_dev, dq_dev, stream);
}

condensa_status condensa_dequantize_bf16(const uint16_t* q_dev, uint64_t n, float* dq_dev, void* stream) {
    return dequantize_impl<CodecBF16>(q_dev, n, dq_dev, stream);
}

condensa_status condensa_profile_read(int phase, double* total_ms, uint64_t* intervals) {
    if (phase < 0 || phase >= CONDENSA_PHASE_COUNT) return CONDENSA_ERR_ARG;
    if (total_ms == nullptr || intervals == nullptr) return CONDENSA_ERR_NULL;
    std::lock_guard<std::mutex> lock(g_prof_mu);
    for (Interval& iv : g_intervals) {
        CONDENSA_HIP(hipEventSynchronize(iv.b));
        float ms = 0.0f;
        CONDENSA_HIP(hipEventElapsedTime(&ms, iv.a, iv.b));
        g_phase_ms[iv.phase] += ms;
        g_phase_n[iv.phase] += 1;
        g_event_pool.push_back(iv.a);
        g_event_pool.push_back(iv.b);
    }
    g_intervals.clear();
    *total_ms = g_phase_ms[phase];
    *intervals = g_phase_n[phase];
    return CONDENSA_OK;
}

condensa_status condensa_profile_reset(void) {
    std::lock_guard<std::mutex> lock(g_prof_mu);
    for (Interval& iv : g_intervals) {
        (void)hipEventSynchronize(iv.b);
        g_event_pool.push_back(iv.a);
        g_event_pool.push_back(iv.b);
    }
    g_intervals.clear();
    for (int i = 0; i < CONDENSA_PHASE_COUNT; ++i) { g_phase_ms[i] = 0.0; g_phase_n[i] = 0; }
    return CONDENSA_OK;
}

condensa_status condensa_lc_sgd_step(const condensa_tensor* tensors, int n_tensors, const float* const* grad_loss,
                                     const float* const* theta, const float* const* lambda,
                                     float* const* momentum_buf, float mu, float lr, float momentum,
                                     void* workspace_dev, size_t workspace_bytes, void* stream,
                                     const condensa_config* config) {
    Config cfg;
    condensa_status rc = resolve_config(config, &cfg);
    if (rc != CONDENSA_OK) return rc;
    if (n_tensors > 0 && (!grad_loss || !theta || !lambda || !momentum_buf)) return CONDENSA_ERR_NULL;
    if (!(mu >= 0.0f) || !std::isfinite(mu) || !std::isfinite(lr) || !std::isfinite(momentum)) return CONDENSA_ERR_DENSITY;
    HostArena arena;
    Tables tb;
    rc = build_tensor_table(tensors, n_tensors, &tb, arena);
    if (rc != CONDENSA_OK) return rc;
    const Layout L = make_layout(CONDENSA_OP_LC_SGD_STEP, tb.N, 0, n_tensors, 1, CONDENSA_SCOPE_GLOBAL, cfg);
    std::vector<OutDesc> out(static_cast<size_t>(n_tensors > 0 ? n_tensors : 1), OutDesc{});
    std::vector<ByteRange> ranges;
    ranges.reserve(static_cast<size_t>(n_tensors) * 5 + 1);
    bool vec = tb.vec;
    for (int t = 0; t < n_tensors; ++t) {
        TensorDesc& d = tb.td[t];
        if (d.n == 0) continue;
        if (!grad_loss[t] || !theta[t] || !lambda[t] || !momentum_buf[t]) return CONDENSA_ERR_NULL;
        d.grad = const_cast<float*>(grad_loss[t]);
        d.lam = lambda[t];
        d.lam_out = momentum_buf[t];
        out[t].theta = const_cast<float*>(theta[t]);
        const void* ptrs[5] = {d.w, d.lam_out, d.grad, d.lam, out[t].theta};
        for (int i = 0; i < 5; ++i) {
            if (!aligned16(ptrs[i])) vec = false;
            ranges.push_back(byte_range(ptrs[i], d.n * 4, i < 2));     // the weights and the momentum buffer are written
        }
    }
    ranges.push_back(byte_range(workspace_dev, workspace_bytes < L.total ? workspace_bytes : L.total, true));
    if (ranges_conflict(ranges.data(), ranges.size())) return CONDENSA_ERR_ARG;
    rc = check_workspace(workspace_dev, workspace_bytes, L);
    if (rc != CONDENSA_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (tb.n_chunks == 0) return CONDENSA_OK;
    const unsigned grid = static_cast<unsigned>(tb.n_chunks * (kChunk / 256));
    bool few = n_tensors <= kSgdFewTensors;                 // chunks are numbered in 32 bits by the launch already
    for (int t = 0; t < n_tensors && few; ++t) few = tb.td[t].n <= 0xFFFFFFFFull;
    if (few) {
        SgdFewArgs f;
        for (int t = 0; t < kSgdFewTensors; ++t) {
            const bool there = t < n_tensors;
            f.w[t] = there ? const_cast<float*>(tb.td[t].w) : nullptr;
            f.grad[t] = there ? tb.td[t].grad : nullptr;
            f.theta[t] = there ? out[t].theta : nullptr;
            f.lam[t] = there ? tb.td[t].lam : nullptr;
            f.mom[t] = there ? tb.td[t].lam_out : nullptr;
            f.n[t] = there ? static_cast<u32>(tb.td[t].n) : 0;
            f.chunk_start[t] = there ? static_cast<u32>(tb.td[t].chunk_start) : ~0u;
        }
        f.mu = mu; f.lr = lr; f.momentum = momentum;
        PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
        if (vec) hipLaunchKernelGGL((k_lc_sgd_few<true>), dim3(grid), dim3(64), 0, st, f);
        else     hipLaunchKernelGGL((k_lc_sgd_few<false>), dim3(grid), dim3(64), 0, st, f);
        CONDENSA_LAUNCH_CHECK();
        return CONDENSA_OK;
    }
    StageImage img;
    rc = begin_call(L, tb, n_tensors, out.data(), out.size(), nullptr, 0, workspace_dev, st, &img);
    if (rc != CONDENSA_OK) return rc;

    DataArgs a{};
    a.td = at<TensorDesc>(workspace_dev, L.td);
    a.chunk_map = at<u32>(workspace_dev, L.chunk_map);
    a.n_chunks = tb.n_chunks;
    a.N = tb.N;
    a.n_tensors = n_tensors;
    a.mu = mu;
    PhaseTimer timer(CONDENSA_PHASE_APPLY, st, cfg);
    const OutDesc* od = at<OutDesc>(workspace_dev, L.out);
    if (vec) hipLaunchKernelGGL((k_lc_sgd<true>), dim3(grid), dim3(64), 0, st, a, od, lr, momentum);
    else     hipLaunchKernelGGL((k_lc_sgd<false>), dim3(grid), dim3(64), 0, st, a, od, lr, momentum);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}

float condensa_mu_schedule(double mu0, double a, int j) { return static_cast<float>(mu0 * std::pow(a, static_cast<double>(j))); }

condensa_status condensa_thin(const float* w_dev, const int64_t* shape, int ndim, const int32_t* keep_out_dev,
                              int64_t n_keep_out, int64_t keep_out_offset, const int32_t* keep_in_dev,
                              int64_t n_keep_in, int64_t keep_in_offset, float* out_dev, void* stream) {
    if (shape == nullptr) return CONDENSA_ERR_NULL;
    if (ndim < 2 || ndim > 4) return CONDENSA_ERR_SHAPE;
    u64 ksize = 1;
    for (int i = 0; i < ndim; ++i) {
        if (shape[i] < 0 || shape[i] > 0x7FFFFFFFll) return CONDENSA_ERR_SHAPE;
        if (i >= 2) ksize *= static_cast<u64>(shape[i]);
    }
    const u64 c_out = static_cast<u64>(shape[0]), c_in = static_cast<u64>(shape[1]);
    if (n_keep_out < 0 || n_keep_in < 0) return CONDENSA_ERR_SIZE;
    const u64 n_out = keep_out_dev ? static_cast<u64>(n_keep_out) : c_out;
    const u64 n_in = keep_in_dev ? static_cast<u64>(n_keep_in) : c_in;
    if (n_out > 0x7FFFFFFFull || n_in > 0x7FFFFFFFull || ksize > 0x7FFFFFFFull) return CONDENSA_ERR_SIZE;
    const u64 total = n_out * n_in * ksize;
    if (total > kMaxElems) return CONDENSA_ERR_SIZE;
    if (total == 0) return CONDENSA_OK;
    if (w_dev == nullptr || out_dev == nullptr) return CONDENSA_ERR_NULL;
    {
        ByteRange r[4] = {byte_range(w_dev, c_out * c_in * ksize * 4, false), byte_range(out_dev, total * 4, true),
                          byte_range(keep_out_dev, keep_out_dev ? n_out * 4 : 0, false),
                          byte_range(keep_in_dev, keep_in_dev ? n_in * 4 : 0, false)};
        if (ranges_conflict(r, 4)) return CONDENSA_ERR_ARG;
    }
    u64 blocks = (total + kBlock - 1) / kBlock;
    if (blocks > 256 * 32) blocks = 256 * 32;
    hipLaunchKernelGGL(k_thin, dim3(static_cast<unsigned>(blocks)), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                       w_dev, c_out, c_in, ksize, keep_out_dev, n_out, keep_out_offset, keep_in_dev, n_in,
                       keep_in_offset, out_dev);
    CONDENSA_LAUNCH_CHECK();
    return CONDENSA_OK;
}

condensa_status condensa_set_option(int option, int64_t value) {
    if (option < 0 || option >= CONDENSA_OPT_COUNT) return CONDENSA_ERR_ARG;
    return set_default_option(option, value);
    return CONDENSA_OK;
}

int64_t condensa_get_option(int option) {
    if (option < 0 || option >= CONDENSA_OPT_COUNT) return -1;
    Config c;
    resolve_config(nullptr, &c);
    return c[option];
}

const char* condensa_status_string(condensa_status s) {
    switch (s) {
        case CONDENSA_OK: return "ok";
        case CONDENSA_ERR_NULL: return "required pointer is NULL";
        case CONDENSA_ERR_SIZE: return "count or size out of range";
        case CONDENSA_ERR_DENSITY: return "density outside [0,1], or mu not finite and positive";
        case CONDENSA_ERR_SHAPE: return "tensor shape not valid for this operator";
        case CONDENSA_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case CONDENSA_ERR_ARG: return "invalid scope, option or aliasing";
        case CONDENSA_ERR_HIP: return "HIP runtime call failed";
        default: return "unknown status";
    }
}

int condensa_last_hip_error(void) { return g_last_hip_error.load(); }

uint64_t condensa_launch_count(void) { return g_launches.load(); }

int condensa_version(void) { return 200; }

void condensa_test_force(unsigned what) { t_force = what; }      // host.h: for tests

}  // extern "C"
