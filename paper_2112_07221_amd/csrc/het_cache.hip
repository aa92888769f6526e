// Host side of the C ABI declared in include/het_cache.h: argument checks, device memory
// owned by the cache, and the kernel sequence of each call.  No step of the method runs on the
// host; the host only decides launch shapes from sizes it already knows (n, max_batch_ids,
// capacity) and never waits for the device inside het_lookup / het_update.
#include "../../include/het_cache.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "cache_kernels.hpp"
#include "key_hash.hpp"
#include "pattern_kernels.hpp"
#include "static_lookup.hpp"

namespace het {          // (compiled in parts of their own)
#define HET_ELSEWHERE(part, ...) extern HET_APPLY_KERNEL(__VA_ARGS__)
HET_APPLY_VARIANTS(HET_ELSEWHERE)
#undef HET_ELSEWHERE
#define HET_ELSEWHERE(part, ...) extern HET_FILL_KERNEL(__VA_ARGS__)
HET_FILL_VARIANTS(HET_ELSEWHERE)
#undef HET_ELSEWHERE
} // namespace het

using namespace het;

// Kernels of the path, as named in profiles and by het_profile_kernel_name.
enum KernelId {
    K_SORT_STAGE, K_PROBE, K_FILL_GATHER, K_APPLY, K_TRIM_STAGE,
    K_TRIM_EVICT, K_DEFERRED_PUSH, K_LINK, K_FLUSH, K_MISC, K_NUM
};
static const char *const kKernelNames[K_NUM] = {
    "sort_stage_kernel", "probe_kernel", "fill_gather_kernel",
    "apply_kernel", "trim_stage_kernel", "trim_evict_kernel", "deferred_push_kernel", "link_kernel", "flush_kernel", "misc"};

struct ProfSpan { int id; hipEvent_t start, stop; };

constexpr int SORT_SETS = 4;
constexpr uint32_t FILL_MAX_BLOCKS = 1024;     // workgroups that fetch missed rows (more only queue up ahead of the gather's)

// A batch announced by het_prefetch: its ids, the buffer set its sort uses and how far the sort has come.
struct Announced {
    const int64_t *ids = nullptr;
    uint32_t n = 0;
    int set = 0;
    int next_stage = 0;              // stages [0, next_stage) are enqueued (carried, or all of them)
};

struct het_cache {
    // creation parameters
    int64_t capacity = 0, s = 0;
    int32_t dim = 0, policy = 0;
    // configuration
    bool configured = false, attached = false;
    bool many = false;               // one of several workers over one global table (het_cache_set_many_writers)
    uint32_t lfu_cap = 16;           // HET_POLICY_LFU_LIGHT: where the use counter stops
    int64_t max_ids = 0;
    int32_t optimizer = 0;
    float eps = 0.f;
    hipStream_t stream = nullptr;
    int location = 0;
    // device state
    CacheView cv{};
    Workspace ws{};
    ApplyBorders bd{};
    TrimPlan tp{};
    // Four sets of sort buffers: the order of the current batch (kept for its update) and up to
    // three batches announced ahead by het_prefetch, whose sorts are carried by the kernels of the
    // calls in between.  (With batches announced two ahead three stand announced when a lookup is called: its own, sorted by
    // then, the next one and the one after that.)
    // Per set the tiles in order of the ranges, [0], and the order, [1].
    uint32_t *keys[SORT_SETS][2] = {}, *idx[SORT_SETS][2] = {};
    uint32_t *sort_words[SORT_SETS] = {};     // SortPlan's cuts and beginnings
    int sort_set = 0;                // the set that holds the current batch's order
    uint32_t sorted_n = 0;           // how many ids that order has (0: there is none yet)
    int older_set = -1;              // the set that still holds the order before it (-1: none does), and how many ids that has
    uint32_t older_n = 0;
    Announced ann[SORT_SETS - 1];    // announced batches, oldest first
    int n_ann = 0;
    TrimPlan sel_tp{};               // the select plan of the rows now cached (fixed at the lookup)
    bool counted = false;            // its rows have been counted (beside the lookup's fetches)
    bool recount = false;            // and which of them hold updates has changed since other than by the update of the batch
    int kept_key_bits = KEPT_BITS;   // width of the policy key the kept histograms were counted for
    bool last_trim_skipped = false;  // the last update had nothing to trim: its evicted-id list is empty
    int cslot = 0;                   // which of the two per-call counter blocks the current call uses
    uint32_t *inv = nullptr;
    uint32_t *tile_free[2] = {nullptr, nullptr};   // free slots per tile, left by a trim; trims alternate between the two
    int tf_last = 0;                 // the one the last trim filled (initially: every slot free)
    uint32_t *ev_ids[2] = {nullptr, nullptr};      // evicted ids of the last two trims, alternating like tile_free
    KeyHash key_hash{};              // the cached keys, if the index of the table's found no room in HBM
    void *index_host = nullptr;      // that index, if neither did
    int max_chunks_per_lane = 1;     // row chunks one lane handles in the apply kernel
    std::vector<void *> owned;       // every device allocation, for destroy
    char *arena = nullptr;           // one allocation that holds all the small arrays side by side (see dev_alloc)
    size_t arena_used = 0;
    // host-backed table: write-back of the last trim's victims still to be enqueued
    bool push_pending = false;
    int push_buf = 0;
    uint32_t push_seq = 0, trim_seq = 0;
    // host-backed table: the stream beside the main one on which rows of the coming batch are fetched
    // ahead and staged rows are written back while the update runs (Section 4.1, 4.2)
    hipStream_t side = nullptr;
    hipEvent_t ev_main = nullptr, ev_link = nullptr;
    bool link_outstanding = false;   // a kernel on that stream has not been waited for yet
    uint32_t pf_serial = 0;
    int pf_slot_next = 0;            // which of the two list counters the next list uses
    struct { bool ready = false; const int64_t *ids = nullptr; uint32_t n = 0, tag = 0; } pf;   // rows fetched ahead, and for which lookup
    // host-side bookkeeping
    uint64_t t_host = 0;             // non-empty lookups so far (equals the device's t)
    bool overflow_pending = false;   // a lookup ran and no trim since
    uint32_t last_lookup_n = 0;
    bool updated = false;            // an update has come since the last lookup
    const int64_t *order_ids = nullptr;   // ids the current sorted order was built from (by a lookup)
    uint32_t order_n = 0;
    bool order_valid = false;
    // optional per-kernel timing (het_profile_begin / het_profile_end)
    bool profiling = false;
    KernelTrace trace[2]{};          // het_profile_trace: the update's kernel, the lookup's second kernel
    // The last lookup left the fetch of its missed keys' rows to the update that reuses its order (table in
    // HBM, one worker): that update reads them from the global table.  Any other call that needs the rows
    // in their slots fetches them first (settle_fetch).
    bool fetch_owed = false;
    uint32_t owed_n = 0, owed_t = 0;
    std::vector<ProfSpan> spans;
};

namespace {

// With HET_DEBUG set in the environment, a failing HIP call is named on stderr.
void report(const char *what, hipError_t e)
{
    if (std::getenv("HET_DEBUG")) std::fprintf(stderr, "[het_cache] %s: %s\n", what, hipGetErrorString(e));
}

#define HIP_TRY(expr)                                  \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) { report(#expr, e_); return HET_EHIP; } \
    } while (0)

// Frees the device allocations made after the first `keep`, and what was taken from the arena after
// `arena_mark` (a call that fails midway leaves nothing behind).
void free_owned_from(het_cache *c, size_t keep, size_t arena_mark)
{
    while (c->owned.size() > keep) {
        if (c->owned.back() == c->arena) { c->arena = nullptr; c->arena_used = 0; }
        (void)hipFree(c->owned.back());
        c->owned.pop_back();
    }
    if (c->arena) c->arena_used = arena_mark;
}

void free_index_host(het_cache *c)
{
    if (c->index_host) (void)hipHostFree(c->index_host);
    c->index_host = nullptr;
}

constexpr size_t ARENA_BYTES = (size_t)128 << 20, ARENA_ITEM_MAX = 8u << 20;

// Arrays of up to 8 MB lie side by side in one allocation of 128 MB; larger ones, and whatever does
// not fit, get their own.  With an allocation per array the probe kernel's time on config 2 depended
// on how many arrays had been allocated before (13.0 or 14.5 us: two more small arrays were enough);
// side by side it does not.
template <typename T>
int dev_alloc(het_cache *c, T **p, size_t count)
{
    const size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
    if (ARENA_BYTES && bytes <= ARENA_ITEM_MAX) {
        if (!c->arena) {
            void *a = nullptr;
            if (hipMalloc(&a, ARENA_BYTES) == hipSuccess) { c->arena = static_cast<char *>(a); c->arena_used = 0; c->owned.push_back(a); }
            else (void)hipGetLastError();
        }
        const size_t at = (c->arena_used + 255) / 256 * 256;
        if (c->arena && at + bytes <= ARENA_BYTES) {
            *p = reinterpret_cast<T *>(c->arena + at);
            c->arena_used = at + bytes;
            return HET_OK;
        }
    }
    void *q = nullptr;
    const hipError_t e = hipMalloc(&q, bytes);
    if (e != hipSuccess) { report("hipMalloc", e); return HET_ENOMEM; }
    c->owned.push_back(q);
    *p = static_cast<T *>(q);
    return HET_OK;
}

inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

inline int bit_width(uint64_t v)
{
    int b = 0;
    while (v) { ++b; v >>= 1; }
    return b;
}

inline uint32_t pow2_at_least(uint64_t v)
{
    uint64_t p = 1;
    while (p < v) p <<= 1;
    return (uint32_t)p;
}

int status_from_bits(uint32_t bits)
{
    if (bits & ERRBIT_RANGE) return HET_ERANGE;
    if (bits & ERRBIT_STATE) return HET_ESTATE;
    return HET_OK;
}

// While profiling, every launch is bracketed by a pair of events on the cache's stream.
struct LaunchScope {
    het_cache *c;
    ProfSpan sp{};
    bool on;
    hipStream_t st;
    LaunchScope(het_cache *cache, int id, hipStream_t stream) : c(cache), on(cache->profiling), st(stream)
    {
        if (!on) return;
        sp.id = id;
        // timing only: no system-scope fence, whose cache write-back would be billed to the kernels
        if (hipEventCreateWithFlags(&sp.start, hipEventDisableSystemFence) != hipSuccess ||
            hipEventCreateWithFlags(&sp.stop, hipEventDisableSystemFence) != hipSuccess) { on = false; return; }
        (void)hipEventRecord(sp.start, st);
    }
    ~LaunchScope()
    {
        if (!on) return;
        (void)hipEventRecord(sp.stop, st);
        c->spans.push_back(sp);
    }
};
#define LAUNCH_ON(cache, stream_, id, ...)         \
    do {                                           \
        LaunchScope scope_(cache, id, stream_);    \
        __VA_ARGS__;                               \
    } while (0)
#define LAUNCH(cache, id, ...) LAUNCH_ON(cache, (cache)->stream, id, __VA_ARGS__)

int launch_ok()
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { report("kernel launch", e); return HET_EHIP; }
    return HET_OK;
}

// Groups of `lanes` threads work on one row; how many 256-thread blocks for `items` rows.
uint32_t row_grid(const RowGeom &g, uint64_t items)
{
    const uint32_t per_block = 256u / (uint32_t)g.lanes;
    return std::max(1u, std::min(cdiv(items, per_block), 256u * 8u));      // at most 8 workgroups per CU
}

// Stage `stage` of the sort of ids[n] into buffer set `set`; carried: its first stage was, or is.  The orders sorted last tell
// where the ranges begin.  (A batch's first stage may read the order that its second one, in a kernel behind it, overwrites.)
SortStage make_stage(het_cache *c, const int64_t *ids, uint32_t n, int set, int stage, bool carried)
{
    SortStage s{};
    SortPlan &sp = s.sp;
    sp.n = n; sp.vocab = c->cv.vocab;
    sp.ranges = sort_ranges(n, carried); sp.ntiles = cdiv(n, SORT_TILE);
    sp.cuts = c->sort_words[set];
    sp.begin = reinterpret_cast<uint16_t *>(sp.cuts + sp.ranges);
    sp.keys = c->keys[set][0]; sp.idx = c->idx[set][0];
    if (c->sorted_n) { sp.known = c->ws.skey; sp.n_known = c->sorted_n; }
    if (c->older_set >= 0) { sp.older = c->keys[c->older_set][1]; sp.n_older = c->older_n; }
    if (set == c->older_set) c->older_set = -1;
    s.ids = ids;
    s.keys_out = c->keys[set][1]; s.idx_out = c->idx[set][1];
    s.stage = stage;
    s.blocks = stage == SORT_PART ? sp.ntiles : sp.ranges;
    return s;
}

SortStage no_stage()
{
    SortStage s{};
    s.stage = -1;
    return s;
}

// Begins a call that touches the cache: per-call counters go to the other counter block.
void begin_call(het_cache *c)
{
    c->cslot = 1 - c->cslot;
    c->cv.last = &c->cv.ds->call[c->cslot];
    c->cv.next_call = &c->cv.ds->call[1 - c->cslot];
}

template <int ITEMS>
void launch_solo(het_cache *c, const int64_t *ids, uint32_t n, int set)
{
    const int bits = std::max(SORT_MIN_BITS, bit_width(c->cv.vocab)), passes = solo_passes(bits, SORT_THREADS_ALONE), width = (bits + passes - 1) / passes;
    LAUNCH(c, K_SORT_STAGE, sort_solo_kernel<ITEMS><<<1, SORT_THREADS_ALONE, solo_lds_bytes(ITEMS, width, SORT_THREADS_ALONE), c->stream>>>(
                                ids, n, c->cv.vocab, passes, width, c->keys[set][1], c->idx[set][1]));
}

// What is left of a sort (stages [first_stage, end)), in kernels of its own.  Up to SOLO_MAX ids none of whose stages has run
// by one workgroup in one launch: its time is the ballots' on one compute unit and grows with the ids (20 bits: 4.9 us
// for 200, 7.7 for 2048, 11.9 for 4096, 19.9 for 8192); two launches take 10.8 us for 3328 ids, 11.7 for 8658.
void sort_now(het_cache *c, const int64_t *ids, uint32_t n, int set, int first_stage)
{
    if (first_stage == 0 && n <= SOLO_MAX) {
        if (set == c->older_set) c->older_set = -1;
        if (n <= SORT_THREADS_ALONE) launch_solo<1>(c, ids, n, set);
        else if (n <= 2 * SORT_THREADS_ALONE) launch_solo<2>(c, ids, n, set);
        else launch_solo<4>(c, ids, n, set);
        return;
    }
    for (int st = first_stage; st < SORT_STAGES; ++st) {
        const SortStage s = make_stage(c, ids, n, set, st, first_stage > 0);
        const uint32_t lds = sort_stage_lds_bytes(s, SORT_THREADS_ALONE);
        if (st == SORT_PART) LAUNCH(c, K_SORT_STAGE, sort_part_kernel<<<s.blocks, SORT_THREADS_ALONE, lds, c->stream>>>(s));
        else LAUNCH(c, K_SORT_STAGE, sort_range_kernel<<<s.blocks, SORT_THREADS_ALONE, lds, c->stream>>>(s));
    }
}

// The next stage of the oldest announced batch whose sort is not complete yet, for the kernel
// that is about to be launched to carry.
SortStage next_ride_of(het_cache *c, int a)
{
    Announced &an = c->ann[a];
    return make_stage(c, an.ids, an.n, an.set, an.next_stage++, true);
}

// What the kernel about to be launched carries: the next stage of the oldest announced batch whose
// sort is not complete yet and, since stages of one sort need a kernel boundary between them, the
// next stage of the batch announced after it.
struct Rides {
    SortStage a, b;
    uint32_t blocks() const { return a.blocks + b.blocks; }
};

// LDS a kernel needs: its own roles' or, if larger, a carried stage's.
uint32_t lds_bytes(size_t own, const Rides &r)
{
    uint32_t need = (uint32_t)own;
    if (r.a.blocks) need = std::max(need, sort_stage_lds_bytes(r.a, SORT_THREADS));
    if (r.b.blocks) need = std::max(need, sort_stage_lds_bytes(r.b, SORT_THREADS));
    return need;
}

// Which kernel is about to be launched: stages of batches of up to LEAVE_MAX ids are left to those that hide them better, if these come
// often enough before the batch is looked up (table in HBM).  With so few ids a lookup's kernels are shorter than a stage's chain.
//   FILL, a lookup's second kernel: leaves them to the updates (if the last call was one; two ahead, a step carried by both
//     kernels and by the updates alone: 400 ids 22.0 and 18.8 us, 4000 27.8 and 26.0, 30000 32.1 and 29.5).
//   READ_TRIM, the eviction of a lookup that follows a lookup: leaves them to the lookups' second kernels, which have two stages of two
//     batches side by side where each kernel had one (lookups only, two ahead: 2000 ids 23.3 and 22.9 us, 8000 24.3 and 22.8, 20000 30.7 and 27.6).
//     The lookup's own batch may be among the announced ones, so the a-th has a of them before it.
enum Carrier { UPDATE, FILL, READ_TRIM };
constexpr uint32_t LEAVE_MAX = 32768;
Rides next_rides(het_cache *c, Carrier who = UPDATE)
{
    Rides r{no_stage(), no_stage()};
    int got = 0;
    for (int a = 0; a < c->n_ann && got < 2; ++a) {
        const int left = SORT_STAGES - c->ann[a].next_stage;
        if (!left) continue;
        const int later = c->side || c->ann[a].n > LEAVE_MAX ? 0 : who == FILL ? (c->updated ? a + 1 : 0) : who == READ_TRIM ? a : 0;
        if (left <= later) continue;
        (got == 0 ? r.a : r.b) = next_ride_of(c, a);
        ++got;
    }
    return r;
}

void drop_oldest_announcement(het_cache *c)
{
    for (int a = 0; a + 1 < c->n_ann; ++a) c->ann[a] = c->ann[a + 1];
    c->n_ann -= 1;
}

void use_order(het_cache *c, int set, uint32_t n)
{
    if (set != c->sort_set && c->sorted_n) { c->older_set = c->sort_set; c->older_n = c->sorted_n; }
    c->sorted_n = n;
    c->sort_set = set;
    c->ws.skey = c->keys[set][1];
    c->ws.perm = c->idx[set][1];
}

// The trim's select plan for the rows cached after the lookup that just ran.
TrimPlan make_trim_plan(const het_cache *c)
{
    TrimPlan tp = c->tp;
    tp.lfu = c->policy == HET_POLICY_LFU || c->policy == HET_POLICY_LFU_LIGHT;
    tp.key_bits = std::max(KEPT_BITS, bit_width(c->t_host));
    tp.passes = tp.key_bits > KEPT_BITS ? 3 : 2;
    tp.t_now = (uint32_t)c->t_host;
    tp.zero_words = (uint32_t)(tp.hist - tp.zero_from) + (tp.passes > 2 ? (uint32_t)SEL_BINS : 0u);
    return tp;
}

// May the rows below and at tau be counted beside the fetches of a lookup?  What holds updates when the trim comes must
// follow from what is known by then.  LRU: rows of the batch are all tied at t_now (see trim_count_body), if they can be victims
// at all.  LFU: a row of the batch that was found has been used twice, unless the light-weight policy stopped counting at 1.
// (Where that held for LRU only up to a capacity of the batch's ids, lookups of 53248 ids over 50000 rows had a kernel for the count, 46.7 us.)
bool count_beside_fill(const het_cache *c, const TrimPlan &tp) { return tp.passes == 2 && !(tp.lfu && c->cv.freq_cap == 1); }

// May the eviction run beside the update?
bool evict_beside_update(const het_cache *c, const TrimPlan &tp)
{
    return count_beside_fill(c, tp) && c->location == HET_BACKING_HBM && !c->many;
}

uint32_t count_blocks(const het_cache *c) { return cdiv(c->cv.n_slots, COUNT_SLOTS); }

constexpr uint32_t STALE_BLOCKS = 128;     // fetch workgroups of a lookup that leaves the missed rows to the update: they refresh the stale rows
constexpr uint32_t PUSH_BLOCKS = 256;      // few workgroups keep the host link full; more only contend
// Workgroups of the kernel that works the host link beside the update: a third of them write back, the others, which mostly
// have more rows to move, fetch ahead (four minibatches and a flush of 106496 ids of 128 floats: 2 691 us with 16 and 16, 2 694
// with 12 and 20, 2 718 with 8 and 24, 2 648 with 16 and 32).
constexpr uint32_t LINK_BLOCKS = 48, LINK_PUSH_BLOCKS = 16;

// Host-backed table: the main stream goes on only when the kernel on the stream beside it is done.
void wait_link(het_cache *c)
{
    if (!c->link_outstanding) return;
    (void)hipStreamWaitEvent(c->stream, c->ev_link, 0);
    c->link_outstanding = false;
}

// Host-backed table: enqueues the write-back a trim left staged, if nobody carried it yet.
void drain_pushes(het_cache *c)
{
    if (!c->push_pending) return;
    wait_link(c);                // (staged copies reach the table in the order they were staged)
    if (c->cv.geom.vec == 4) LAUNCH(c, K_DEFERRED_PUSH, deferred_push_kernel<4><<<PUSH_BLOCKS, 256, 0, c->stream>>>(c->cv, c->push_buf));
    else LAUNCH(c, K_DEFERRED_PUSH, deferred_push_kernel<1><<<PUSH_BLOCKS, 256, 0, c->stream>>>(c->cv, c->push_buf));
    c->push_pending = false;
}

// A lookup left the fetch of its missed keys' rows to the update that reuses its order, and that
// update is not what comes next: fetch them now (the lookup's lists are still in place: nothing
// has sorted, probed or trimmed since).
template <int VEC>
int settle_fetch_impl(het_cache *c)
{
    const uint32_t n = c->owed_n, ptiles = cdiv(n, PT_TILE);
    const uint32_t fill_blocks = std::min(cdiv(row_grid(c->cv.geom, n), (uint32_t)FILL_ROWS), FILL_MAX_BLOCKS);
    const TrimPlan none{};
    const SortStage no = no_stage();
    LAUNCH(c, K_FILL_GATHER, fill_gather_kernel<VEC, false, false, false><<<fill_blocks, 256, sizeof(FillLds), c->stream>>>(
                                 c->cv, c->ws, n, c->owed_t, ptiles, fill_blocks, none, 0u, nullptr, nullptr, 0u, nullptr, no, no,
                                 0u, 0, 0u, Ahead{}, KernelTrace{}, 2, 1u));
    c->fetch_owed = false;
    return launch_ok();
}
int settle_fetch(het_cache *c)
{
    if (!c->fetch_owed) return HET_OK;
    return c->cv.geom.vec == 4 ? settle_fetch_impl<4>(c) : settle_fetch_impl<1>(c);
}

// Where the key index found no room in HBM, kernels of their own search, fill and clear the hash table of the cached
// keys (key_hash.hpp): the slots of a sorted order's keys, before a kernel asks for them; the keys a lookup has
// fetched; the keys a trim has dropped.
void hash_find(het_cache *c, const uint32_t *skey, uint32_t n)
{
    if (!c->key_hash.entries) return;
    LAUNCH(c, K_MISC, key_find_kernel<<<cdiv(n, 256), 256, 0, c->stream>>>(c->key_hash, skey, n, c->cv.vocab, c->cv.slot_of));
}
void hash_insert(het_cache *c, uint32_t n)
{
    if (!c->key_hash.entries) return;
    LAUNCH(c, K_MISC, key_insert_kernel<<<cdiv(n, 256), 256, 0, c->stream>>>(c->key_hash, c->ws.skey, c->ws.cls, c->ws.head_slot, n, c->cv.vocab));
}
void hash_erase(het_cache *c, const TrimPlan &tp)
{
    if (!c->key_hash.entries) return;
    LAUNCH(c, K_MISC, key_erase_kernel<<<cdiv(c->last_lookup_n, 256), 256, 0, c->stream>>>(c->key_hash, tp.ev_ids, &c->cv.ds->ev_n[tp.ev_slot]));
}

// The plan of the eviction about to be launched: which of the alternating arrays it fills.
TrimPlan plan_eviction(het_cache *c, bool fetched_dirty)
{
    TrimPlan tp = c->sel_tp;
    const int fill = 1 - c->tf_last;                 // the idle array: cleared by the lookup in between
    tp.fetched_dirty = fetched_dirty;
    tp.tile_free = c->tile_free[fill];
    tp.ev_slot = fill;
    tp.ev_ids = c->ev_ids[fill];
    tp.push_seq = ++c->trim_seq;
    if (c->trim_seq == 0x7FFFFFFFu) c->trim_seq = 0;        // 0 means "none", the top bit marks lists of keys fetched ahead; a wrap is harmless (see HostLink::pend)
    c->tf_last = fill;
    c->overflow_pending = false;
    c->last_trim_skipped = false;
    c->order_valid = false;          // slots recorded for the sorted order may be gone now
    return tp;
}

uint32_t evict_grid(const het_cache *c) { return cdiv(c->cv.n_slots, EV_SLOTS) + 1; }        // (the last one keeps the histograms)

// Evict(): the rows below and at tau are counted, if no kernel carried that, then the eviction itself.
// updated: the batch of the lookup that left the overflow has been updated since, by its own order.
template <int VEC>
int run_trim(het_cache *c, bool counted, bool updated)
{
    drain_pushes(c);                                 // the staging buffers alternate: the one before last must be gone
    if (counted && c->recount) {
        LAUNCH(c, K_TRIM_STAGE, clear_words_kernel<<<1, 256, 0, c->stream>>>(c->sel_tp.zero_from, (uint32_t)(c->sel_tp.hist - c->sel_tp.zero_from)));
        counted = false;
    }
    if (!counted) LAUNCH(c, K_TRIM_STAGE, trim_stage_kernel<<<count_blocks(c), TRIM_THREADS, 0, c->stream>>>(c->cv, c->sel_tp));
    const TrimPlan tp = plan_eviction(c, counted && c->counted && updated);
    const Rides ride = next_rides(c, c->updated ? UPDATE : READ_TRIM);
    const uint32_t ev_blocks = evict_grid(c);
    // Rows of a kilobyte or more: the pushes run at the memory's limit, and a fourth workgroup per
    // compute unit only gets in the others' way (config 5: 107 us against 97).  Asking for more LDS
    // than a quarter of a compute unit's keeps it to three.  Not where the update pushes the rows it
    // fetches early: then few victims are left to copy, and the fourth workgroup pays (config 5:
    // 25.9 -> 23.5 us).
    const uint32_t lds_floor = c->cv.geom.lanes == 64 && VEC == 4 && !c->cv.early_cc ? 44u * 1024u : 0u;
    const uint32_t lds = std::max(lds_bytes(sizeof(EvictLds), ride), lds_floor);
    if (c->many)
        LAUNCH(c, K_TRIM_EVICT, trim_evict_kernel<VEC, true, true><<<ride.blocks() + ev_blocks, TRIM_THREADS, lds, c->stream>>>(c->cv, tp, ride.a, ride.b));
    else if (ride.blocks())
        LAUNCH(c, K_TRIM_EVICT, trim_evict_kernel<VEC, true, false><<<ride.blocks() + ev_blocks, TRIM_THREADS, lds, c->stream>>>(c->cv, tp, ride.a, ride.b));
    else
        LAUNCH(c, K_TRIM_EVICT, trim_evict_kernel<VEC, false, false><<<ev_blocks, TRIM_THREADS, lds, c->stream>>>(c->cv, tp, ride.a, ride.b));
    hash_erase(c, tp);
    if (c->location == HET_BACKING_PINNED_HOST) { c->push_pending = true; c->push_buf = tp.ev_slot; c->push_seq = tp.push_seq; }
    return launch_ok();
}

// Row groups that add up one bag of a pooled lookup together: as many as fit a workgroup and fill the chip's places (half its
// threads; the kernel has registers for that many), with four rows each on average.  One group a bag left most of the chip idle
// and waited for the longest bag: 1001 bags of 0 to 150 rows of 100 floats 68.9 -> 55.5 us a step, 1000 of 100 rows of 16 floats
// 87.9 -> 53.3, 2048 of 200 rows of 256 floats 235.9 -> 234.3; two rows each: 8000 bags of 5 rows 48.6 -> 51.4.
constexpr uint64_t POOL_THREADS = 262144;
constexpr uint32_t POOL_SHARE = 4;
uint32_t pool_split(const RowGeom &g, uint32_t n, uint32_t n_bags)
{
    uint32_t split = 1;
    while (2 * split * (uint32_t)g.lanes <= 256u && (uint64_t)n_bags * 2 * split * (uint32_t)g.lanes <= POOL_THREADS && n >= (uint64_t)POOL_SHARE * n_bags * 2 * split) split *= 2;
    return split;
}

template <int VEC>
int run_lookup(het_cache *c, const int64_t *ids, uint32_t n, const int64_t *offsets, uint32_t n_bags, float *out)
{
    begin_call(c);
    c->t_host += 1;
    int rc;
    if ((rc = settle_fetch(c)) != HET_OK) return rc;
    if (c->overflow_pending && (rc = run_trim<VEC>(c, c->counted, false)) != HET_OK) return rc;   // a Read that follows a Read
    // The sorted order: announced by het_prefetch and sorted inside the kernels launched since
    // (what is left of it runs now), or sorted here.  Announcements older than the one used are
    // void; with no match they all stand (a later lookup may still use them).
    int match = -1;
    for (int a = 0; a < c->n_ann && match < 0; ++a)
        if (c->ann[a].ids == ids && c->ann[a].n == n) match = a;
    if (match >= 0) {
        for (int a = 0; a < match; ++a) drop_oldest_announcement(c);
        const Announced an = c->ann[0];
        drop_oldest_announcement(c);
        sort_now(c, ids, n, an.set, an.next_stage);
        use_order(c, an.set, n);
    } else {
        sort_now(c, ids, n, c->sort_set, 0);             // over the previous batch's order: it is not needed any more
        use_order(c, c->sort_set, n);
    }
    const uint32_t t_now = (uint32_t)c->t_host;
    const uint32_t split = offsets ? pool_split(c->cv.geom, n, n_bags) : 1u;
    if (c->cv.direct) {
        // no cache: mark the runs, then gather straight from the global table
        const uint32_t dtiles = cdiv(n, PT_TILE), dblocks = dtiles * (match >= 0 ? 2u : 1u);
        LAUNCH(c, K_PROBE, direct_probe_kernel<true><<<dblocks, PT_THREADS, 0, c->stream>>>(c->cv, c->ws, n, t_now, dtiles, match >= 0 ? ids : nullptr, offsets ? c->inv : nullptr));
        const Rides ride = next_rides(c, FILL);
        const uint32_t grid = ride.blocks() + row_grid(c->cv.geom, offsets ? (uint64_t)n_bags * split : cdiv(n, GATHER_ROWS));
        const uint32_t lds = lds_bytes(std::max(sizeof(FillLds), sizeof(TrimLds)), ride);
        const TrimPlan none{};
#define GATHER_ONLY_T(POOLED, RIDE, TRACE)                                                                               \
    LAUNCH(c, K_FILL_GATHER, fill_gather_kernel<VEC, POOLED, RIDE, TRACE><<<grid, 256, lds, c->stream>>>(                   \
                                 c->cv, c->ws, n, t_now, 0u, 0u, none, 0u, out, offsets, n_bags, c->inv, ride.a, ride.b, 0u, 0, 0u, Ahead{}, c->trace[1], 0, split))
#define GATHER_ONLY(POOLED, RIDE) do { if (c->trace[1].rec) GATHER_ONLY_T(POOLED, RIDE, true); else GATHER_ONLY_T(POOLED, RIDE, false); } while (0)
        if (!offsets) { if (ride.blocks()) GATHER_ONLY(false, true); else GATHER_ONLY(false, false); }
        else { if (ride.blocks()) GATHER_ONLY(true, true); else GATHER_ONLY(true, false); }
#undef GATHER_ONLY
#undef GATHER_ONLY_T
        if ((rc = launch_ok()) != HET_OK) return rc;
        c->updated = false;
        c->last_lookup_n = n;
        c->order_ids = ids; c->order_n = n; c->order_valid = true;
        return HET_OK;
    }
    const uint32_t ptiles = cdiv(n, PT_TILE), stiles = cdiv(c->cv.n_slots, PT_TILE);
    // The select plan of the trim that follows this lookup.
    c->sel_tp = make_trim_plan(c);
    const TrimPlan &tp = c->sel_tp;
    if (tp.key_bits != c->kept_key_bits) {           // (iterations 2^22, 2^23, ...: wider bins)
        LAUNCH(c, K_TRIM_STAGE, clear_words_kernel<<<1024, 256, 0, c->stream>>>(tp.coarse, KEPT_WORDS));
        LAUNCH(c, K_TRIM_STAGE, kept_recount_kernel<<<std::min(cdiv(c->cv.n_slots, TRIM_THREADS), 1024u), TRIM_THREADS, 0, c->stream>>>(c->cv, tp));
        c->kept_key_bits = tp.key_bits;
    }
    {
        hash_find(c, c->ws.skey, n);
        const uint32_t blocks = ptiles + (match >= 0 ? ptiles : 0u) + stiles;
        LAUNCH(c, K_PROBE, probe_kernel<true><<<blocks, PT_THREADS, 0, c->stream>>>(
                               c->cv, c->ws, n, t_now, ptiles, c->tile_free[c->tf_last], c->tile_free[1 - c->tf_last], (uint32_t)(1 - c->tf_last),
                               tp, match >= 0 ? ids : nullptr, c->side ? c->pf_slot_next : -1, offsets ? c->inv : nullptr));
    }

    c->counted = count_beside_fill(c, tp);
    c->recount = false;
    const uint32_t hist_blocks = c->counted ? count_blocks(c) : (tp.passes > 2 ? std::min(cdiv(c->cv.n_slots, TRIM_TILE), 1024u) : 0u);
    const uint32_t fill_blocks = std::min(cdiv(row_grid(c->cv.geom, n), (uint32_t)FILL_ROWS), FILL_MAX_BLOCKS);     // they come first: theirs is the longer chain
    const uint32_t lds_own = (uint32_t)std::max(sizeof(FillLds), sizeof(TrimLds));
#define FILL_GATHER_T(POOLED, RIDE, TRACE, GRID, FILLB, HISTB, PUSHB)                                                     \
    LAUNCH(c, K_FILL_GATHER, fill_gather_kernel<VEC, POOLED, RIDE, TRACE><<<GRID, 256, lds_bytes(lds_own, ride), c->stream>>>( \
                                 c->cv, c->ws, n, t_now, ptiles, FILLB, tp, HISTB, out, offsets, n_bags, c->inv, ride.a, ride.b, \
                                 PUSHB, c->push_buf, c->push_seq, ah, c->trace[1], fetch_mode, split))
#define FILL_GATHER(POOLED, RIDE, GRID, FILLB, HISTB, PUSHB)                                                              \
    do {                                                                                                                  \
        if (c->trace[1].rec) FILL_GATHER_T(POOLED, RIDE, true, GRID, FILLB, HISTB, PUSHB);                                \
        else FILL_GATHER_T(POOLED, RIDE, false, GRID, FILLB, HISTB, PUSHB);                                               \
    } while (0)
#define FILL_GATHER_ANY(GRID, FILLB, HISTB, PUSHB)                                                                        \
    do {                                                                                                                  \
        if (!offsets) {                                                                                                   \
            if (ride.blocks()) FILL_GATHER(false, true, GRID, FILLB, HISTB, PUSHB);                                       \
            else FILL_GATHER(false, false, GRID, FILLB, HISTB, PUSHB);                                                    \
        } else {                                                                                                          \
            if (ride.blocks()) FILL_GATHER(true, true, GRID, FILLB, HISTB, PUSHB);                                        \
            else FILL_GATHER(true, false, GRID, FILLB, HISTB, PUSHB);                                                     \
        }                                                                                                                 \
    } while (0)
    const uint32_t gather_blocks = row_grid(c->cv.geom, offsets ? (uint64_t)n_bags * split : cdiv(n, GATHER_ROWS));
    Ahead ah{};
    int fetch_mode = 0;
    if (c->location == HET_BACKING_HBM && !c->many) {
        // one kernel: the gather reads a missed key's row from the global table, beside the fetch.
        // The missed keys' rows themselves are left to the update that is expected to follow (it reads
        // them from the global table and writes them to their slots with its step applied); the fetch
        // workgroups that remain refresh the stale rows.
        // Row-wise Adagrad: only if an update came since the lookup before; where lookups follow lookups the rows left would take a kernel
        // of their own (settle_fetch): lookups alone of 3000 ids of 64 floats 32.5 us, 27.3 with the rows fetched here.
        const Rides ride = next_rides(c, FILL);
        const bool owe = !c->cv.rowwise || c->updated;
        fetch_mode = owe ? 1 : 0;
        const uint32_t fb = owe ? std::min(fill_blocks, STALE_BLOCKS) : fill_blocks;
        FILL_GATHER_ANY(ride.blocks() + fb + ptiles + hist_blocks + gather_blocks, fb, hist_blocks, 0u);
        if (owe) { c->fetch_owed = true; c->owed_n = n; c->owed_t = t_now; }
        hash_insert(c, n);
    } else {
        // Host-backed table: the fetches come over the host link, and the last trim's write-back
        // goes the other way in the same kernel; the gather follows and reads the cached copies.
        // Several workers: a row that is synchronised takes a new value (the server's row plus this
        // worker's push), which the gather must see, so it follows in a launch of its own too.
        // Host-backed table with a batch announced for the next lookup: the second kernel lists that
        // batch's keys that are not cached, and a kernel on the stream beside this one brings their rows
        // into HBM while the update runs, with the write-back going the other way beside them (so the
        // fetch kernel leaves the write-back to it); the next lookup's fetch kernel finds them there.
        const bool host = c->side != nullptr;
        Announced *next = host && c->n_ann > 0 ? &c->ann[0] : nullptr;
        if (host) {
            // rows fetched ahead for this lookup; and no refresh of this lookup may overtake an older staged copy
            wait_link(c);
            if (c->pf.ready && c->pf.ids == ids && c->pf.n == n) ah.use_tag = c->pf.tag;
            c->pf.ready = false;
        }
        const uint32_t push_blocks = c->push_pending && !next ? PUSH_BLOCKS : 0u;
        const uint32_t fetch_blocks = c->location == HET_BACKING_HBM ? fill_blocks : std::min(fill_blocks, PUSH_BLOCKS);
        {
            const Rides ride = next_rides(c, FILL);
            FILL_GATHER_ANY(ride.blocks() + push_blocks + fetch_blocks + ptiles + hist_blocks, fetch_blocks, hist_blocks, push_blocks);
        }
        if (push_blocks) c->push_pending = false;
        hash_insert(c, n);
        ah = Ahead{};
        if (next) {
            sort_now(c, next->ids, next->n, next->set, next->next_stage);                                // what is left of its sort runs now
            next->next_stage = SORT_STAGES;
            c->pf_serial = (c->pf_serial % 0x7FFFFFFFu) + 1;
            ah.skey = c->keys[next->set][1];
            ah.n = next->n;
            ah.blocks = cdiv(next->n, 256);
            ah.list_tag = 0x80000000u | c->pf_serial;
            ah.list_slot = c->pf_slot_next;
            ah.pending_seq = c->push_pending ? c->push_seq : 0u;
            hash_find(c, ah.skey, ah.n);
        }
        {
            const Rides ride = next_rides(c, FILL);
            FILL_GATHER_ANY(ride.blocks() + ah.blocks + gather_blocks, 0u, 0u, 0u);
        }
        if (next) {
            if ((rc = launch_ok()) != HET_OK) return rc;
            HIP_TRY(hipEventRecord(c->ev_main, c->stream));
            HIP_TRY(hipStreamWaitEvent(c->side, c->ev_main, 0));
            const int pbuf = c->push_pending ? c->push_buf : -1;
            // Few workgroups with several rows in flight each: a compute unit that waits for the host link
            // serves its other waves' memory requests behind those that wait, so every compute unit that
            // hosts a workgroup of this kernel is slow for the update's kernels meanwhile (measured: with
            // 512 workgroups the optimizer step took as long as the whole transfer).
            if (VEC == 4) LAUNCH_ON(c, c->side, K_LINK, link_kernel<4><<<LINK_BLOCKS, 256, 0, c->side>>>(c->cv, pbuf, ah.list_slot, c->push_buf, LINK_PUSH_BLOCKS));
            else LAUNCH_ON(c, c->side, K_LINK, link_kernel<1><<<LINK_BLOCKS, 256, 0, c->side>>>(c->cv, pbuf, ah.list_slot, c->push_buf, LINK_PUSH_BLOCKS));
            if ((rc = launch_ok()) != HET_OK) return rc;
            HIP_TRY(hipEventRecord(c->ev_link, c->side));
            c->link_outstanding = true;
            c->push_pending = false;
            c->pf.ready = true; c->pf.ids = next->ids; c->pf.n = next->n; c->pf.tag = ah.list_tag;
            c->pf_slot_next ^= 1;
        }
    }
#undef FILL_GATHER_ANY
#undef FILL_GATHER
#undef FILL_GATHER_T
    if ((rc = launch_ok()) != HET_OK) return rc;
    c->overflow_pending = true;
    c->updated = false;
    c->last_lookup_n = n;
    c->order_ids = ids; c->order_n = n; c->order_valid = true;
    return HET_OK;
}

// The kernel of Write.  Where the rows below and at tau could not be counted beside the lookup's fetches it
// carries that count in extra workgroups.  The count looks at the clocks the kernel is moving, which is sound
// only when the update is known to touch exactly the rows the last Read touched (it reuses that Read's order): see
// TrimPlan::dirty_stamp.
// Where they were counted there, the eviction runs beside the update (see evict_body) if the update is the one the lookup left
// its fetches to (c->fetch_owed: table in HBM, one worker): rows it touches that are victims it
// writes to the global table itself, instead of to their slots.
// `trim`: a trim follows.  Returns whether its rows have been counted.
template <int VEC, int MAXC, int TILE, bool EARLY, int OPT>
bool launch_apply_opt(het_cache *c, bool verify, const int64_t *ids, uint32_t n, const float *grads, const int64_t *offsets, uint32_t n_bags, float lr,
                      bool trim)
{
    const uint32_t grid = cdiv(n, TILE);
    TrimPlan tp = c->sel_tp;
    bool counted = c->counted;
    const int fresh = verify && c->fetch_owed ? 1 : 0;          // (verify: this update reuses the lookup's order)
    if (fresh) c->fetch_owed = false;
    const bool evict = trim && fresh && !c->recount && evict_beside_update(c, tp) && !c->profiling;      // (per-kernel timing: in a kernel of its own, to tell the two apart)
    uint32_t extra = 0;
    if (evict) { tp = plan_eviction(c, true); extra = evict_grid(c); }
    else if (trim && !counted && verify && c->cv.freq_cap != 1) {    // (light-weight LFU with a cap of 1 leaves rows of the batch unstamped that can be evicted; with a larger cap those it leaves unstamped cannot)
        extra = count_blocks(c); counted = true; tp.dirty_stamp = (uint32_t)c->t_host;
    }
    const Rides ride = next_rides(c);
    const uint32_t lds = lds_bytes(std::max({sizeof(TrimLds), sizeof(EvictLds), sizeof(ApplyLds<VEC, TILE>)}), ride);
#define APPLY(MODE)                                                                                                                              \
    LAUNCH(c, K_APPLY, apply_kernel<VEC, MAXC, MODE, TILE, EARLY, OPT><<<ride.blocks() + grid + extra + (verify ? cdiv(n, VERIFY_TILE) : 0u), AP_THREADS, lds, c->stream>>>( \
                           c->cv, c->ws, c->bd, ids, grads, offsets, n_bags, lr, c->eps, n, grid, tp, extra, ride.a, ride.b, c->trace[0], fresh))
    if (evict) {
        if (!tp.lfu && (int64_t)n > c->capacity) APPLY(AP_REUSED_EVICT_TIED); else APPLY(AP_REUSED_EVICT);
        hash_erase(c, tp);
    } else if (verify) APPLY(AP_REUSED); else APPLY(AP_SORTED);
#undef APPLY
    return counted;
}

template <int VEC, int MAXC, int TILE, bool EARLY>
bool launch_apply_early(het_cache *c, bool verify, const int64_t *ids, uint32_t n, const float *grads, const int64_t *offsets, uint32_t n_bags, float lr,
                        bool trim)
{
    if constexpr (MAXC > 1) return launch_apply_opt<VEC, MAXC, TILE, EARLY, AO_ANY>(c, verify, ids, n, grads, offsets, n_bags, lr, trim);
    else {
        if constexpr (!EARLY)            // (row-wise Adagrad does not push early)
            if (c->cv.rowwise) return launch_apply_opt<VEC, MAXC, TILE, EARLY, AO_ROWWISE>(c, verify, ids, n, grads, offsets, n_bags, lr, trim);
        return c->cv.adagrad ? launch_apply_opt<VEC, MAXC, TILE, EARLY, AO_ADAGRAD>(c, verify, ids, n, grads, offsets, n_bags, lr, trim)
                             : launch_apply_opt<VEC, MAXC, TILE, EARLY, AO_SGD>(c, verify, ids, n, grads, offsets, n_bags, lr, trim);
    }
}

// EARLY: the variant that also pushes the rows it fetches (CacheView::early_cc in use).
template <int VEC, int MAXC, int TILE>
bool launch_apply_tile(het_cache *c, bool verify, const int64_t *ids, uint32_t n, const float *grads, const int64_t *offsets, uint32_t n_bags, float lr,
                      bool trim)
{
    if constexpr (VEC == 4)          // (only rows of whole 16-byte pieces push early)
        if (c->cv.early_cc) return launch_apply_early<VEC, MAXC, TILE, true>(c, verify, ids, n, grads, offsets, n_bags, lr, trim);
    return launch_apply_early<VEC, MAXC, TILE, false>(c, verify, ids, n, grads, offsets, n_bags, lr, trim);
}

template <int VEC, int MAXC>
bool launch_apply(het_cache *c, bool verify, const int64_t *ids, uint32_t n, const float *grads, const int64_t *offsets, uint32_t n_bags, float lr,
                 bool trim)
{
    // rows of more than 128 floats (64 lanes to a row) have one row piece per lane or more; narrower ones exactly one
    if constexpr (MAXC == 1)
        if (ap_tile_for(c->cv.geom.lanes) == 64) return launch_apply_tile<VEC, MAXC, 64>(c, verify, ids, n, grads, offsets, n_bags, lr, trim);
    return launch_apply_tile<VEC, MAXC, 128>(c, verify, ids, n, grads, offsets, n_bags, lr, trim);
}

template <int VEC>
int run_update(het_cache *c, const int64_t *ids, uint32_t n, const int64_t *offsets, uint32_t n_bags,
               const float *grads, float lr)
{
    begin_call(c);
    int rc;
    c->updated = true;
    // The ids of the preceding lookup, passed again: reuse its sorted order (the apply kernel
    // checks every id against it).  Anything else is sorted and probed afresh, into the current
    // set of sort buffers (announced batches use the other sets).
    const bool reuse = c->order_valid && ids == c->order_ids && n == c->order_n;
    if (!reuse) {
        if ((rc = settle_fetch(c)) != HET_OK) return rc;
        sort_now(c, ids, n, c->sort_set, 0);
        use_order(c, c->sort_set, n);
        if (c->cv.direct)
            LAUNCH(c, K_PROBE, direct_probe_kernel<false><<<cdiv(n, PT_TILE), PT_THREADS, 0, c->stream>>>(c->cv, c->ws, n, (uint32_t)c->t_host, cdiv(n, PT_TILE), nullptr, nullptr));
        else {
            hash_find(c, c->ws.skey, n);
            LAUNCH(c, K_PROBE, probe_kernel<false><<<cdiv(n, PT_TILE), PT_THREADS, 0, c->stream>>>(
                                   c->cv, c->ws, n, (uint32_t)c->t_host, cdiv(n, PT_TILE), nullptr, nullptr, 0u, TrimPlan{}, nullptr, -1, nullptr));
        }
    }
    // Only a lookup leaves rows above capacity; an update that follows no lookup has nothing to trim.
    const bool trim = c->overflow_pending;
    bool counted = false;
    switch (c->max_chunks_per_lane) {
    case 1: counted = launch_apply<VEC, 1>(c, reuse, ids, n, grads, offsets, n_bags, lr, trim); break;
    case 2: counted = launch_apply<VEC, 2>(c, reuse, ids, n, grads, offsets, n_bags, lr, trim); break;
    case 4: counted = launch_apply<VEC, 4>(c, reuse, ids, n, grads, offsets, n_bags, lr, trim); break;
    default: counted = launch_apply<VEC, 16>(c, reuse, ids, n, grads, offsets, n_bags, lr, trim); break;
    }
    if ((rc = launch_ok()) != HET_OK) return rc;
    if (!trim) { c->last_trim_skipped = true; c->order_valid = false; return HET_OK; }
    if (!reuse) c->recount = true;               // rows counted as clean may hold updates now
    if (!c->overflow_pending) return HET_OK;         // (evicted beside the update)
    return run_trim<VEC>(c, counted, reuse);
}

int sync_all(het_cache *c)
{
    drain_pushes(c);
    if (c->side) HIP_TRY(hipStreamSynchronize(c->side));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return HET_OK;
}

int sync_and_status(het_cache *c, DState *host_copy)
{
    int rc0 = sync_all(c);
    if (rc0) return rc0;
    DState h;
    HIP_TRY(hipMemcpy(&h, c->cv.ds, sizeof(DState), hipMemcpyDeviceToHost));
    if (host_copy) *host_copy = h;
    return status_from_bits(h.err);
}

void to_public(const Counters &in, het_counters *out)
{
    out->n = (int64_t)in.n; out->unique = (int64_t)in.unique; out->hit = (int64_t)in.hit;
    out->stale = (int64_t)in.stale; out->miss = (int64_t)in.miss; out->evicted = (int64_t)in.evicted;
    out->evicted_dirty = (int64_t)in.evicted_dirty; out->stale_dirty = (int64_t)in.stale_dirty;
    out->flushed = (int64_t)in.flushed;
}

bool ready(const het_cache *c) { return c && c->configured && c->attached; }

// het_lookup_nocache_static.  Ids up to this many are checked by one workgroup inside the gather's
// launch (two rounds of loads: 0.4 us longer than without a check at 4096 ids); beyond it that
// workgroup would outlast the gather, and a launch of its own (1.5 us) clears err_bits first.
constexpr uint32_t STATIC_CHECK_MAX = 2 * STATIC_CHECK_LOADS * STATIC_THREADS;

template <int VEC>
void launch_static(const RowGeom &g, const float *table, uint32_t vocab, const int64_t *ids, uint32_t n, float *out,
                   uint32_t *err_bits, hipStream_t stream)
{
    const uint32_t blocks = cdiv(n, STATIC_THREADS / (uint32_t)g.lanes);
    if (err_bits && n <= STATIC_CHECK_MAX) {
        static_lookup_kernel<VEC, true><<<blocks + 1, STATIC_THREADS, 0, stream>>>(table, vocab, g, ids, n, out, err_bits);
        return;
    }
    if (err_bits) static_clear_kernel<<<1, 1, 0, stream>>>(err_bits);
    static_lookup_kernel<VEC, false><<<blocks, STATIC_THREADS, 0, stream>>>(table, vocab, g, ids, n, out, err_bits);
}

} // namespace

extern "C" {

int het_cache_create(het_cache **out, int64_t capacity, int32_t dim, int64_t s, int32_t policy)
{
    if (!out || capacity <= 0 || dim <= 0 || s < 0) return HET_EINVAL;
    if (policy != HET_POLICY_LRU && policy != HET_POLICY_LFU && policy != HET_POLICY_NONE && policy != HET_POLICY_LFU_LIGHT) return HET_EINVAL;
    if (capacity >= (1ll << 30) || dim > (1 << 20)) return HET_EINVAL;
    het_cache *c = new (std::nothrow) het_cache();
    if (!c) return HET_ENOMEM;
    c->capacity = capacity; c->dim = dim; c->s = s; c->policy = policy;
    *out = c;
    return HET_OK;
}

static int configure_impl(het_cache *c, int64_t max_batch_ids, int32_t optimizer, float eps, void *hip_stream)
{
    if (!c || c->configured || max_batch_ids <= 0 || max_batch_ids > (int64_t)MAX_PROBE_TILES * PT_TILE) return HET_EINVAL;
    if (optimizer != HET_OPT_SGD && optimizer != HET_OPT_ADAGRAD && optimizer != HET_OPT_ADAGRAD_ROWWISE) return HET_EINVAL;
    if (!(eps >= 0.f)) return HET_EINVAL;
    if (optimizer == HET_OPT_ADAGRAD_ROWWISE && c->many) return HET_EINVAL;
    c->max_ids = max_batch_ids; c->optimizer = optimizer; c->eps = eps;
    c->stream = static_cast<hipStream_t>(hip_stream);

    CacheView &cv = c->cv;
    const bool direct = c->policy == HET_POLICY_NONE;       // no cache: rows and accumulators are the global table's (set at attach)
    cv.direct = direct;
    const uint64_t P = direct ? 1 : (uint64_t)c->capacity + (uint64_t)max_batch_ids;
    cv.n_slots = (uint32_t)P; cv.capacity = (uint32_t)c->capacity; cv.max_ids = (uint32_t)max_batch_ids;
    cv.s = c->s; cv.adagrad = optimizer == HET_OPT_ADAGRAD; cv.rowwise = optimizer == HET_OPT_ADAGRAD_ROWWISE;
    RowGeom g;
    g.dim = c->dim; g.vec = (c->dim % 4 == 0) ? 4 : 1; g.chunks = c->dim / g.vec;
    g.lanes = (int)std::min<uint32_t>(64u, pow2_at_least((uint64_t)g.chunks));
    cv.geom = g;
    const int per_lane = (g.chunks + g.lanes - 1) / g.lanes;
    c->max_chunks_per_lane = per_lane <= 1 ? 1 : (per_lane <= 2 ? 2 : (per_lane <= 4 ? 4 : 16));
    if (per_lane > 16) return HET_EINVAL;               // rows wider than 64 lanes x 16 chunks
    if (cv.rowwise && per_lane > 1) return HET_EINVAL;  // row-wise Adagrad: the row group holds the whole row's gradient at once

    int rc = HET_OK;
    const size_t row_elems = (size_t)P * (size_t)c->dim;
    if (!direct && (rc = dev_alloc(c, &cv.rows, row_elems))) return rc;
    if (!direct && cv.adagrad && (rc = dev_alloc(c, &cv.acc, row_elems))) return rc;
    if (!direct && cv.rowwise && (rc = dev_alloc(c, &cv.acc, (size_t)P))) return rc;
    cv.many = c->many;
    // Early push where rows have more than 64 floats, in whole 16-byte pieces (measured: rows of 128 floats 1.4 %,
    // of 256 floats 6 % faster; with rows of 64 floats the update loses what the eviction gains).
    if (!direct && !c->many && !cv.rowwise && g.vec == 4 && g.lanes >= 32) {          // (dropped again at attach if the table is behind the host link)
        if ((rc = dev_alloc(c, &cv.early_cc, (size_t)P))) return rc;
        HIP_TRY(hipMemsetAsync(cv.early_cc, 0, (size_t)P * sizeof(uint32_t), c->stream));
    }
    cv.freq_cap = c->policy == HET_POLICY_LFU_LIGHT ? c->lfu_cap : 0u;
    if (c->many && (rc = dev_alloc(c, &cv.rows0, row_elems))) return rc;
    if (c->many && cv.adagrad && (rc = dev_alloc(c, &cv.acc0, row_elems))) return rc;
    if ((rc = dev_alloc(c, &cv.slot_key, P)) || (rc = dev_alloc(c, &cv.meta, P))) return rc;
    if ((rc = dev_alloc(c, &cv.free_list, (size_t)max_batch_ids)) || (rc = dev_alloc(c, &cv.was_free, P))) return rc;
    if ((rc = dev_alloc(c, &cv.ds, 1))) return rc;
    // workspaces
    Workspace &ws = c->ws;
    const size_t N = (size_t)max_batch_ids;
    const size_t ptiles = cdiv(N, PT_TILE);
    const size_t ap_tiles = cdiv(N, (per_lane <= 1 ? ap_tile_for(g.lanes) : 128));
    for (int set = 0; set < SORT_SETS; ++set) {
        for (int i = 0; i < 2; ++i)
            if ((rc = dev_alloc(c, &c->keys[set][i], N)) || (rc = dev_alloc(c, &c->idx[set][i], N))) return rc;
        if ((rc = dev_alloc(c, &c->sort_words[set], sort_plan_words((uint32_t)N)))) return rc;
    }
    c->cv.last = &cv.ds->call[0];
    c->cv.next_call = &cv.ds->call[1];
    if ((rc = dev_alloc(c, &ws.src, N)) || (rc = dev_alloc(c, &ws.head_slot, N)) || (rc = dev_alloc(c, &ws.cls, N)) ||
        (rc = dev_alloc(c, &ws.tile_miss, ptiles)) || (rc = dev_alloc(c, &ws.tile_stale, ptiles)) || (rc = dev_alloc(c, &ws.tile_hit, ptiles)) ||
        (rc = dev_alloc(c, &ws.miss_stage, ptiles * PT_TILE)) || (rc = dev_alloc(c, &ws.stale_stage, ptiles * PT_TILE)) ||
        (rc = dev_alloc(c, &c->inv, N)) || (rc = dev_alloc(c, &ws.bag_of, N)) ||
        (rc = dev_alloc(c, &c->bd.part, ap_tiles * 4 * (size_t)c->dim)) || (rc = dev_alloc(c, &c->bd.slot, ap_tiles)) ||      // (tiles' sums, then groups' sums: see ApplyBorders)
        (rc = dev_alloc(c, &c->bd.arrived, ap_tiles * 3)) || (rc = dev_alloc(c, &c->bd.from_key, ap_tiles)))
        return rc;
    const size_t slot_tiles = cdiv(P, TRIM_TILE), ev_blocks = cdiv(P, EV_SLOTS), ev_supers = cdiv(ev_blocks, EV_SUPER);
    // the counts per EV_SUPER eviction blocks, and the third digit's histogram behind them
    if ((rc = dev_alloc(c, &c->tp.zero_from, 4 * ev_supers + SEL_BINS)) || (rc = dev_alloc(c, &c->tp.blk_cnt, ev_blocks)) ||
        (rc = dev_alloc(c, &c->tp.coarse, direct ? 1 : (size_t)KEPT_WORDS)) ||
        (rc = dev_alloc(c, &c->tile_free[0], slot_tiles)) ||
        (rc = dev_alloc(c, &c->tile_free[1], slot_tiles)) || (rc = dev_alloc(c, &c->ev_ids[0], P)) || (rc = dev_alloc(c, &c->ev_ids[1], P)))
        return rc;
    c->tp.sup_cnt = reinterpret_cast<uint4 *>(c->tp.zero_from);
    c->tp.hist = c->tp.zero_from + 4 * ev_supers;
    c->tp.fine = c->tp.coarse + SEL_BINS;
    if (!direct) HIP_TRY(hipMemsetAsync(c->tp.coarse, 0, (size_t)KEPT_WORDS * sizeof(uint32_t), c->stream));
    {   // before the first trim every slot is free
        std::vector<uint32_t> full(slot_tiles);
        for (size_t t = 0; t < slot_tiles; ++t) full[t] = (uint32_t)std::min<uint64_t>(TRIM_TILE, P - t * TRIM_TILE);
        HIP_TRY(hipMemcpy(c->tile_free[0], full.data(), slot_tiles * sizeof(uint32_t), hipMemcpyHostToDevice));
    }
    HIP_TRY(hipMemsetAsync(c->tile_free[1], 0, slot_tiles * sizeof(uint32_t), c->stream));

    // the sort's own kernels ask for more LDS than a launch gets unasked
    const int max_lds = 144 * 1024;      // (of 160: some of it is taken by the compiler)
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&sort_part_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, max_lds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&sort_range_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, max_lds));
    HIP_TRY(hipMemsetAsync(c->bd.arrived, 0, ap_tiles * 3 * sizeof(uint32_t), c->stream));
    HIP_TRY(hipMemsetAsync(cv.ds, 0, sizeof(DState), c->stream));
    init_cache_kernel<<<1024, 256, 0, c->stream>>>(cv);
    if ((rc = launch_ok())) return rc;
    HIP_TRY(hipStreamSynchronize(c->stream));
    c->configured = true;
    return HET_OK;
}

int het_cache_configure(het_cache *c, int64_t max_batch_ids, int32_t optimizer, float eps, void *hip_stream)
{
    const size_t keep = c ? c->owned.size() : 0, mark = c ? c->arena_used : 0;
    const int rc = configure_impl(c, max_batch_ids, optimizer, eps, hip_stream);
    if (rc != HET_OK && c && !c->configured) free_owned_from(c, keep, mark);     // a retry starts from nothing
    return rc;
}

// The hash table of the cached keys, and where its searches leave their answers.
static int alloc_key_hash(het_cache *c)
{
    KeyHash &h = c->key_hash;
    const uint32_t buckets = pow2_at_least(cdiv((uint64_t)c->cv.n_slots * 4, BUCKET_ENTRIES));
    const size_t keep = c->owned.size(), mark = c->arena_used;
    int rc;
    if ((rc = dev_alloc(c, &h.entries, (size_t)buckets * BUCKET_ENTRIES)) || (rc = dev_alloc(c, &h.reach, buckets)) ||
        (rc = dev_alloc(c, &c->cv.slot_of, (size_t)c->max_ids))) {
        free_owned_from(c, keep, mark);
        h.entries = nullptr;
        return rc;
    }
    h.mask = buckets - 1;
    h.shift = 64 - (bit_width(buckets) - 1);
    static_assert(ENTRY_EMPTY == ~0ull, "filled byte by byte");
    HIP_TRY(hipMemsetAsync(h.entries, 0xFF, (size_t)buckets * BUCKET_ENTRIES * sizeof(uint64_t), c->stream));
    HIP_TRY(hipMemsetAsync(h.reach, 0, (size_t)buckets * sizeof(uint32_t), c->stream));
    return HET_OK;
}

// Find's index, nothing cached yet: 4 bytes per row of the table; if HBM has no room for them (a table that fills it),
// a hash table of the size of the cache; if not even for that, the former in pinned host memory.
static int alloc_index(het_cache *c, int64_t vocab)
{
    const size_t bytes = (size_t)vocab * sizeof(int32_t);
    c->cv.by_position = 0;
    c->key_hash.entries = nullptr;
    if (dev_alloc(c, &c->cv.slot_of, (size_t)vocab) != HET_OK) {
        (void)hipGetLastError();
        const int rc = alloc_key_hash(c);
        if (rc != HET_ENOMEM) { c->cv.by_position = 1; return rc; }
        (void)hipGetLastError();
        if (hipHostMalloc(&c->index_host, bytes, hipHostMallocDefault) != hipSuccess) { (void)hipGetLastError(); c->index_host = nullptr; return HET_ENOMEM; }
        c->cv.slot_of = static_cast<int32_t *>(c->index_host);
    }
    static_assert(SLOT_NONE == -1, "filled byte by byte");
    HIP_TRY(hipMemsetAsync(c->cv.slot_of, 0xFF, bytes, c->stream));
    return HET_OK;
}

static int attach_impl(het_cache *c, float *table, float *state, uint32_t *cg, int64_t vocab, int32_t location)
{
    if (!c || !c->configured || !table || !cg || vocab <= 0 || vocab >= 0xFFFFFFFFll) return HET_EINVAL;
    if (location != HET_BACKING_HBM && location != HET_BACKING_PINNED_HOST) return HET_EINVAL;
    if (c->optimizer != HET_OPT_SGD && !state) return HET_EINVAL;
    if (c->optimizer == HET_OPT_ADAGRAD_ROWWISE && location != HET_BACKING_HBM) return HET_EINVAL;
    if (c->attached) return HET_EINVAL;
    if (c->many && location != HET_BACKING_HBM) return HET_EINVAL;      // several workers: the shared table lives in HBM
    if (location == HET_BACKING_PINNED_HOST) {
        // kernels need the device-side alias of the mapped host memory
        void *dt = nullptr, *dst = nullptr, *dcg = nullptr;
        HIP_TRY(hipHostGetDevicePointer(&dt, table, 0));
        HIP_TRY(hipHostGetDevicePointer(&dcg, cg, 0));
        if (state) HIP_TRY(hipHostGetDevicePointer(&dst, state, 0));
        table = static_cast<float *>(dt); cg = static_cast<uint32_t *>(dcg); state = static_cast<float *>(dst);
    }
    c->cv.W = table; c->cv.A = state; c->cv.Cg = cg; c->cv.Cg_host = nullptr; c->cv.vocab = (uint32_t)vocab;
    if (c->cv.direct) {
        if (vocab >= (1ll << 31)) return HET_EINVAL;        // a key stands for its own slot
        c->cv.rows = table; c->cv.acc = state;
    } else if (location == HET_BACKING_PINNED_HOST) {
        // The kernels work on a mirror of the global clocks in HBM (a probe must not cross the host
        // link for four bytes per key); the caller's array is written through.  Evicted rows are
        // staged in HBM and written back behind the step (HostLink).
        int rc;
        uint32_t *mirror = nullptr;
        if ((rc = dev_alloc(c, &mirror, (size_t)vocab))) return rc;
        HIP_TRY(hipMemcpy(mirror, cg, (size_t)vocab * sizeof(uint32_t), hipMemcpyDefault));
        c->cv.Cg_host = cg;
        c->cv.Cg = mirror;
        c->cv.early_cc = nullptr;            // (no early push over the host link: the update does not fetch there)
        HostLink &hl = c->cv.hl;
        const size_t N = (size_t)c->max_ids, row_elems = N * (size_t)c->dim;
        if ((rc = dev_alloc(c, &hl.pend, (size_t)vocab))) return rc;
        HIP_TRY(hipMemset(hl.pend, 0, (size_t)vocab * sizeof(uint64_t)));
        for (int b = 0; b < 2; ++b) {
            if ((rc = dev_alloc(c, &hl.rows[b], row_elems)) || (rc = dev_alloc(c, &hl.keys[b], N)) || (rc = dev_alloc(c, &hl.cg[b], N))) return rc;
            if (state && (rc = dev_alloc(c, &hl.acc[b], row_elems))) return rc;
        }
        if ((rc = dev_alloc(c, &hl.pf_rows, row_elems)) || (rc = dev_alloc(c, &hl.pf_keys, N)) || (rc = dev_alloc(c, &hl.pf_from, N))) return rc;
        if (state && (rc = dev_alloc(c, &hl.pf_acc, row_elems))) return rc;
        // the stream beside the main one (default priority), and the two events that order them
        HIP_TRY(hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
        HIP_TRY(hipEventCreateWithFlags(&c->ev_main, hipEventDisableTiming));
        HIP_TRY(hipEventCreateWithFlags(&c->ev_link, hipEventDisableTiming));
    }
    if (!c->cv.direct) {                 // last: the only array that can do without HBM
        const int rc = alloc_index(c, vocab);
        if (rc) return rc;
    }
    c->location = location;
    c->attached = true;
    return HET_OK;
}

int het_attach_backing(het_cache *c, float *table, float *state, uint32_t *cg, int64_t vocab, int32_t location)
{
    const size_t keep = c ? c->owned.size() : 0, mark = c ? c->arena_used : 0;
    const bool was = c && c->attached;
    const int rc = attach_impl(c, table, state, cg, vocab, location);
    if (rc != HET_OK && c && !was) {
        free_owned_from(c, keep, mark);
        free_index_host(c);
        if (c->ev_main) { (void)hipEventDestroy(c->ev_main); c->ev_main = nullptr; }
        if (c->ev_link) { (void)hipEventDestroy(c->ev_link); c->ev_link = nullptr; }
        if (c->side) { (void)hipStreamDestroy(c->side); c->side = nullptr; }
    }
    return rc;
}

int het_cache_set_lfu_cap(het_cache *c, uint32_t cap)
{
    if (!c || c->configured || c->policy != HET_POLICY_LFU_LIGHT || cap == 0) return HET_EINVAL;
    c->lfu_cap = cap;
    return HET_OK;
}

int het_cache_set_many_writers(het_cache *c)
{
    if (!c || c->configured || c->policy == HET_POLICY_NONE) return HET_EINVAL;
    c->many = true;
    return HET_OK;
}

int het_cache_set_iteration(het_cache *c, int64_t iteration)
{
    if (!ready(c) || c->overflow_pending || iteration < (int64_t)c->t_host || iteration >= (1ll << 32) - (1ll << 20)) return HET_EINVAL;
    c->t_host = (uint64_t)iteration;             // (the device takes it from the next lookup, which widens the kept histograms' bins if it must)
    return HET_OK;
}

int het_backing_foreign_update(het_cache *c, const int64_t *ids, const float *deltas, int64_t n)
{
    if (!ready(c) || n < 0 || n >= (1ll << 31) || c->location != HET_BACKING_HBM) return HET_EINVAL;
    if (n == 0) return HET_OK;
    if (!ids || !deltas) return HET_EINVAL;
    const uint32_t grid = row_grid(c->cv.geom, (uint64_t)n);
    if (c->cv.geom.vec == 4) LAUNCH(c, K_MISC, foreign_update_kernel<4><<<grid, 256, 0, c->stream>>>(c->cv, ids, deltas, (uint32_t)n));
    else LAUNCH(c, K_MISC, foreign_update_kernel<1><<<grid, 256, 0, c->stream>>>(c->cv, ids, deltas, (uint32_t)n));
    return launch_ok();
}

int het_prefetch_cancel(het_cache *c)
{
    if (!c || !c->configured) return HET_EINVAL;
    // stages already enqueued read their buffer in stream order before anything enqueued from now on;
    // stages not enqueued yet never will be
    c->n_ann = 0;
    c->pf.ready = false;             // rows fetched ahead for a withdrawn batch are not used
    return HET_OK;
}

int het_prefetch(het_cache *c, const int64_t *ids, int64_t n)
{
    if (!ready(c) || n < 0 || n > c->max_ids) return HET_EINVAL;
    if (n == 0) return HET_OK;
    if (!ids) return HET_EINVAL;
    // Nothing is launched here: the kernels of the calls that follow carry the sort, stage by
    // stage, into a buffer set that neither the current order nor an earlier announcement uses.
    // With every spare set taken, the oldest announcement makes room.
    if (c->n_ann && c->ann[c->n_ann - 1].ids == ids && c->ann[c->n_ann - 1].n == (uint32_t)n) return HET_OK;   // said already
    if (c->n_ann == SORT_SETS - 1) drop_oldest_announcement(c);
    for (int set = 0; set < SORT_SETS; ++set) {
        bool taken = set == c->sort_set;
        for (int a = 0; a < c->n_ann; ++a) taken = taken || c->ann[a].set == set;
        if (taken) continue;
        Announced an;
        an.ids = ids; an.n = (uint32_t)n; an.set = set; an.next_stage = 0;
        c->ann[c->n_ann++] = an;
        break;
    }
    return HET_OK;
}

int het_lookup(het_cache *c, const int64_t *ids, int64_t n, float *out)
{
    if (!ready(c) || n < 0 || n > c->max_ids) return HET_EINVAL;
    if (n == 0) return HET_OK;
    if (!ids || !out) return HET_EINVAL;
    return c->cv.geom.vec == 4 ? run_lookup<4>(c, ids, (uint32_t)n, nullptr, 0, out)
                               : run_lookup<1>(c, ids, (uint32_t)n, nullptr, 0, out);
}

int het_lookup_pooled(het_cache *c, const int64_t *ids, int64_t n, const int64_t *offsets, int64_t n_bags, float *out)
{
    if (!ready(c) || n < 0 || n > c->max_ids) return HET_EINVAL;
    if (n == 0) return HET_OK;
    if (!ids || !out || !offsets || n_bags <= 0 || n_bags >= (1ll << 31)) return HET_EINVAL;
    return c->cv.geom.vec == 4 ? run_lookup<4>(c, ids, (uint32_t)n, offsets, (uint32_t)n_bags, out)
                               : run_lookup<1>(c, ids, (uint32_t)n, offsets, (uint32_t)n_bags, out);
}

int het_update(het_cache *c, const int64_t *ids, const float *grads, int64_t n, float lr)
{
    if (!ready(c) || n < 0 || n > c->max_ids) return HET_EINVAL;
    if (n == 0) return HET_OK;
    if (!ids || !grads) return HET_EINVAL;
    return c->cv.geom.vec == 4 ? run_update<4>(c, ids, (uint32_t)n, nullptr, 0, grads, lr)
                               : run_update<1>(c, ids, (uint32_t)n, nullptr, 0, grads, lr);
}

int het_update_pooled(het_cache *c, const int64_t *ids, int64_t n, const int64_t *offsets, const float *bag_grads,
                      int64_t n_bags, float lr)
{
    if (!ready(c) || n < 0 || n > c->max_ids) return HET_EINVAL;
    if (n == 0) return HET_OK;
    if (!ids || !bag_grads || !offsets || n_bags <= 0 || n_bags >= (1ll << 31)) return HET_EINVAL;
    return c->cv.geom.vec == 4 ? run_update<4>(c, ids, (uint32_t)n, offsets, (uint32_t)n_bags, bag_grads, lr)
                               : run_update<1>(c, ids, (uint32_t)n, offsets, (uint32_t)n_bags, bag_grads, lr);
}

int het_flush(het_cache *c)
{
    if (!ready(c)) return HET_EINVAL;
    begin_call(c);
    c->n_ann = 0;                // announcements do not outlive a flush
    c->recount = true;           // (rows counted as holding updates hold none afterwards)
    c->pf.ready = false;
    wait_link(c);                // (nothing the flush writes may be overtaken by an older staged copy)
    drain_pushes(c);             // (a staged copy of a row reaches the table before anything the flush writes)
    { int rc0 = settle_fetch(c); if (rc0) return rc0; }
    const uint32_t grid = row_grid(c->cv.geom, c->cv.n_slots);
    if (c->cv.geom.vec == 4) LAUNCH(c, K_FLUSH, flush_kernel<4><<<grid, 256, 0, c->stream>>>(c->cv));
    else LAUNCH(c, K_FLUSH, flush_kernel<1><<<grid, 256, 0, c->stream>>>(c->cv));
    int rc = launch_ok();
    if (rc) return rc;
    return sync_and_status(c, nullptr);
}

int het_stats(het_cache *c, het_stats_t *out)
{
    if (!c || !c->configured || !out) return HET_EINVAL;
    DState h;
    int rc = sync_and_status(c, &h);
    if (rc == HET_EHIP) return rc;
    to_public(h.call[c->cslot], &out->last);
    to_public(h.total, &out->total);
    // between a lookup and its update the overflow is still cached; after a trim the count is the capacity at most
    out->resident = c->overflow_pending ? h.size : std::min<int64_t>(h.size, c->capacity);
    out->iteration = h.t;
    out->error_bits = (int32_t)h.err;
    return HET_OK;
}

int het_clear_error(het_cache *c)
{
    if (!c || !c->configured) return HET_EINVAL;
    { int rc0 = sync_all(c); if (rc0) return rc0; }
    HIP_TRY(hipMemset(&c->cv.ds->err, 0, sizeof(uint32_t)));
    return HET_OK;
}

int het_export_state(het_cache *c, int64_t *keys, int32_t *slots, uint32_t *cs, uint32_t *cc, uint32_t *last_use,
                     uint32_t *freq, int64_t *n_resident)
{
    if (!c || !c->configured) return HET_EINVAL;
    { int rc0 = sync_all(c); if (rc0) return rc0; }
    const size_t P = c->cv.n_slots;
    std::vector<uint32_t> k(P);
    std::vector<SlotMeta> m(P);
    HIP_TRY(hipMemcpy(k.data(), c->cv.slot_key, P * 4, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(m.data(), c->cv.meta, P * sizeof(SlotMeta), hipMemcpyDeviceToHost));
    int64_t r = 0;
    for (size_t slot = 0; slot < P; ++slot) {
        if (k[slot] == KEY_NONE) continue;
        if (keys) keys[r] = k[slot];
        if (slots) slots[r] = (int32_t)slot;
        if (cs) cs[r] = m[slot].cs;
        if (cc) cc[r] = m[slot].cc;
        if (last_use) last_use[r] = m[slot].last_use;
        if (freq) freq[r] = m[slot].freq;
        ++r;
    }
    if (n_resident) *n_resident = r;
    return HET_OK;
}

int het_export_rows(het_cache *c, float *rows, float *acc)
{
    if (!c || !c->configured) return HET_EINVAL;
    { int rc0 = settle_fetch(c); if (rc0) return rc0; }
    { int rc0 = sync_all(c); if (rc0) return rc0; }
    const size_t P = c->cv.n_slots, D = (size_t)c->dim;
    if (c->cv.direct) return HET_OK;                 // no cache: nothing is ever cached
    std::vector<uint32_t> k(P);
    HIP_TRY(hipMemcpy(k.data(), c->cv.slot_key, P * 4, hipMemcpyDeviceToHost));
    // the slot arrays come over in a few large copies (a copy per row would be one synchronous
    // transfer per cached row) and are compacted here
    const size_t step = std::max<size_t>(1, ((size_t)64 << 20) / (D * 4));
    std::vector<float> buf(std::min(step, P) * D);
    for (int which = 0; which < 2; ++which) {
        float *dst = which ? acc : rows;
        const float *src = which ? c->cv.acc : c->cv.rows;
        if (!dst || !src) continue;
        const size_t W = which && c->cv.rowwise ? 1 : D;        // (row-wise Adagrad: one accumulator per row)
        size_t r = 0;
        for (size_t s0 = 0; s0 < P; s0 += step) {
            const size_t cnt = std::min(step, P - s0);
            bool any = false;
            for (size_t i = 0; i < cnt && !any; ++i) any = k[s0 + i] != KEY_NONE;
            if (!any) continue;
            HIP_TRY(hipMemcpy(buf.data(), src + s0 * W, cnt * W * 4, hipMemcpyDeviceToHost));
            for (size_t i = 0; i < cnt; ++i)
                if (k[s0 + i] != KEY_NONE) { std::memcpy(dst + r * W, buf.data() + i * W, W * 4); ++r; }
        }
    }
    return HET_OK;
}

int het_last_lookup(het_cache *c, int64_t *keys, int32_t *cls, int32_t *slots, int64_t *n_unique)
{
    if (!c || !c->configured) return HET_EINVAL;
    { int rc0 = sync_all(c); if (rc0) return rc0; }
    const size_t n = c->last_lookup_n;
    std::vector<uint32_t> k(n);
    std::vector<int32_t> sl(n);
    std::vector<uint8_t> cl(n);
    if (n) {
        HIP_TRY(hipMemcpy(k.data(), c->ws.skey, n * 4, hipMemcpyDeviceToHost));
        HIP_TRY(hipMemcpy(sl.data(), c->ws.head_slot, n * 4, hipMemcpyDeviceToHost));
        HIP_TRY(hipMemcpy(cl.data(), c->ws.cls, n, hipMemcpyDeviceToHost));
    }
    int64_t u = 0;
    for (size_t j = 0; j < n; ++j) {             // per-key facts sit at the head of each run
        if (k[j] == c->cv.vocab || (j > 0 && k[j] == k[j - 1])) continue;
        if (keys) keys[u] = k[j];
        if (cls) cls[u] = cl[j];
        if (slots) slots[u] = sl[j];
        ++u;
    }
    if (n_unique) *n_unique = u;
    return HET_OK;
}

int het_last_evicted(het_cache *c, int64_t *ids, int64_t *n)
{
    if (!c || !c->configured) return HET_EINVAL;
    { int rc0 = sync_all(c); if (rc0) return rc0; }
    DState h;
    HIP_TRY(hipMemcpy(&h, c->cv.ds, sizeof(DState), hipMemcpyDeviceToHost));
    const int last = c->tf_last;                         // the list the last trim filled
    const uint32_t ev_n = c->last_trim_skipped ? 0u : h.ev_n[last];
    std::vector<uint32_t> e(ev_n);
    if (ev_n) HIP_TRY(hipMemcpy(e.data(), c->ev_ids[last], (size_t)ev_n * 4, hipMemcpyDeviceToHost));
    for (size_t i = 0; i < e.size(); ++i)
        if (ids) ids[i] = e[i];
    if (n) *n = (int64_t)ev_n;
    return HET_OK;
}

// ---- a Read without a cache object and without any allocation ------------------------------
int het_lookup_nocache_static(const float *table, int64_t vocab, int32_t dim, const int64_t *ids, int64_t n, float *out,
                              uint32_t *err_bits, void *hip_stream)
{
    if (n < 0 || n > (int64_t)HET_NOALLOC_MAX_IDS || dim <= 0 || vocab <= 0 || vocab >= (1ll << 31)) return HET_EINVAL;
    if (n == 0) return HET_OK;
    if (!table || !ids || !out) return HET_EINVAL;
    RowGeom g;
    g.dim = dim; g.vec = (dim % 4 == 0) ? 4 : 1; g.chunks = dim / g.vec;
    g.lanes = (int)std::min<uint32_t>(64u, pow2_at_least((uint64_t)g.chunks));
    if ((g.chunks + g.lanes - 1) / g.lanes > 16) return HET_EINVAL;          // rows wider than the kernels take
    const hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (g.vec == 4) launch_static<4>(g, table, (uint32_t)vocab, ids, (uint32_t)n, out, err_bits, st);
    else launch_static<1>(g, table, (uint32_t)vocab, ids, (uint32_t)n, out, err_bits, st);
    return launch_ok();
}

int het_profile_begin(het_cache *c)
{
    if (!c || !c->configured || c->profiling) return HET_EINVAL;
    c->profiling = true;
    return HET_OK;
}

int het_profile_end(het_cache *c, double *total_ms, int64_t *launches, int32_t n_kernels)
{
    if (!c || !c->profiling) return HET_EINVAL;
    c->profiling = false;
    int rc = HET_OK;
    if (sync_all(c) != HET_OK) rc = HET_EHIP;
    for (int i = 0; i < n_kernels; ++i) {
        if (total_ms) total_ms[i] = 0.0;
        if (launches) launches[i] = 0;
    }
    for (ProfSpan &sp : c->spans) {
        float ms = 0.f;
        if (rc == HET_OK && hipEventElapsedTime(&ms, sp.start, sp.stop) == hipSuccess && sp.id < n_kernels) {
            if (total_ms) total_ms[sp.id] += ms;
            if (launches) launches[sp.id] += 1;
        }
        (void)hipEventDestroy(sp.start);
        (void)hipEventDestroy(sp.stop);
    }
    c->spans.clear();
    return rc;
}

int het_profile_rows(int32_t pattern, float *x, float *a, const float *src, const uint32_t *idx, int64_t n, int32_t dim,
                     const uint32_t *gidx, int32_t per, int32_t reps, double *avg_ms, void *hip_stream)
{
    if (pattern < 0 || pattern > 2 || n <= 0 || n > (int64_t)1 << 30 || dim <= 0 || dim % 4 || reps <= 0 || !avg_ms || !x) return HET_EINVAL;
    if (pattern != HET_PATTERN_UPDATE && !src) return HET_EINVAL;
    if (pattern != HET_PATTERN_COPY && !idx) return HET_EINVAL;
    if (pattern == HET_PATTERN_UPDATE && (per < 0 || per > 3 || per == 1 || (per > 0 && (!src || !gidx)))) return HET_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    const int lanes = std::min(dim / 4, 64);
    if (lanes & (lanes - 1)) return HET_EINVAL;          // (row groups of 1, 2, 4, ... 64 lanes: rows of 4, 8, 16, ... 128 floats, or wider)
    const uint32_t per_block = 256u / (uint32_t)lanes;
    const uint32_t rows_at_once = pattern == HET_PATTERN_UPDATE ? PAT_UPDATE_ROWS : PAT_ROWS;
    const uint32_t grid = std::max(1u, std::min(cdiv(cdiv((uint64_t)n, rows_at_once), per_block), 256u * 8u));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_TRY(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return HET_EHIP; }
    int rc = HET_OK;
    for (int rep = -2; rep < reps && rc == HET_OK; ++rep) {          // (two launches first that are not timed)
        if (rep == 0 && hipEventRecord(e0, st) != hipSuccess) rc = HET_EHIP;
        if (pattern == HET_PATTERN_UPDATE && per == 0) pattern_update_kernel<0><<<grid, 256, 0, st>>>(x, a, idx, (uint32_t)n, dim, nullptr, nullptr);
        else if (pattern == HET_PATTERN_UPDATE && per == 2) pattern_update_kernel<2><<<grid, 256, 0, st>>>(x, a, idx, (uint32_t)n, dim, src, gidx);
        else if (pattern == HET_PATTERN_UPDATE) pattern_update_kernel<3><<<grid, 256, 0, st>>>(x, a, idx, (uint32_t)n, dim, src, gidx);
        else pattern_gather_kernel<<<grid, 256, 0, st>>>(src, x, pattern == HET_PATTERN_GATHER ? idx : nullptr, (uint32_t)n, dim);
        if (hipGetLastError() != hipSuccess) rc = HET_EHIP;
    }
    float ms = 0.f;
    if (rc == HET_OK && (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                         hipEventElapsedTime(&ms, e0, e1) != hipSuccess)) rc = HET_EHIP;
    (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
    *avg_ms = (double)ms / reps;
    return rc;
}

int het_profile_trace(het_cache *c, int32_t kernel, uint64_t *records, int64_t capacity)
{
    if (!c || !c->configured || capacity < 0 || capacity > (int64_t)1 << 24 || (capacity > 0 && !records)) return HET_EINVAL;
    if (kernel != K_APPLY && kernel != K_FILL_GATHER) return HET_EINVAL;
    KernelTrace &t = c->trace[kernel == K_APPLY ? 0 : 1];
    t.rec = capacity ? reinterpret_cast<unsigned long long *>(records) : nullptr;
    t.cap = (uint32_t)capacity;
    return HET_OK;
}

int het_profile_kernel_count(void) { return K_NUM; }

const char *het_profile_kernel_name(int index) { return index >= 0 && index < K_NUM ? kKernelNames[index] : ""; }

int het_cache_destroy(het_cache *c)
{
    if (!c) return HET_OK;
    int rc = HET_OK;
    if (c->configured && sync_all(c) != HET_OK) rc = HET_EHIP;
    if (c->ev_main) (void)hipEventDestroy(c->ev_main);
    if (c->ev_link) (void)hipEventDestroy(c->ev_link);
    if (c->side) (void)hipStreamDestroy(c->side);
    for (void *p : c->owned)
        if (hipFree(p) != hipSuccess) rc = HET_EHIP;
    free_index_host(c);
    delete c;
    return rc;
}

#ifndef HET_BUILD_ID
#define HET_BUILD_ID "unknown"
#endif
const char *het_build_id(void) { return HET_BUILD_ID; }

const char *het_strerror(int status)
{
    switch (status) {
    case HET_OK: return "ok";
    case HET_EINVAL: return "invalid argument or call order";
    case HET_ENOMEM: return "out of memory";
    case HET_EHIP: return "HIP runtime error";
    case HET_ERANGE: return "an id was outside [0, vocab)";
    case HET_ESTATE: return "update of an id that is not cached";
    default: return "unknown status";
    }
}

} // extern "C"
