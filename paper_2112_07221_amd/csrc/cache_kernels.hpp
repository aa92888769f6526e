// Kernels of the cache step proper: Read (Algorithm 2 of the paper), Write (Algorithm 3), the
// policy trim Evict() (Section 3.1, Section 4.3) and flush.
//
// Device-side counts never travel to the host inside a call.  Where a kernel needs the number
// of items an earlier kernel found in other tiles (misses, stale rows, free slots, rows tied at
// the eviction threshold), the earlier kernel leaves one count per tile and the later kernel
// adds up the counts of the tiles before its own: "count at the producer, prefix at the
// consumer".  That keeps every ordering decision (which miss takes which free slot, which of
// several equal policy keys is evicted) a function of sorted order alone, never of the arrival
// order of atomics, and no workgroup ever waits for another.
#pragma once
#include "common.hpp"
#include "sort_unique.hpp"

namespace het {

// Clocks (Section 3.1) and policy counters (Section 4.3) of one cache slot; read and written
// as one 16-byte word where several fields are needed.
struct alignas(16) SlotMeta {
    uint32_t cs;         // start clock c_s
    uint32_t cc;         // local clock c_c
    uint32_t last_use;   // iteration of the last Read that had the key
    uint32_t freq;       // number of Reads that had the key since it was fetched
};
__device__ __forceinline__ uint4 load_meta(const SlotMeta *m, uint32_t slot) { return reinterpret_cast<const uint4 *>(m)[slot]; }
__device__ __forceinline__ void store_meta(SlotMeta *m, uint32_t slot, uint32_t cs, uint32_t cc, uint32_t lu, uint32_t fr)
{
    reinterpret_cast<uint4 *>(m)[slot] = make_uint4(cs, cc, lu, fr);
}

// A global table in pinned host memory is written behind the step: a trim copies the rows it
// evicts (those that hold updates) into a staging buffer in HBM, and the copy over the host link
// travels inside the next Read's fetch kernel, where it shares the link, which is full duplex,
// with the fetches going the other way.  `pend` lets a fetch find a row that is still on its way.
struct HostLink {
    float *rows[2], *acc[2];      // staging, [max_ids][dim] each; trims alternate between the two
    uint32_t *keys[2], *cg[2];    // per staged row: its key and the global clock it will carry
    uint64_t *pend;               // [vocab]: (serial number of the trim << 32) | staging index of the key's staged row,
                                  // or (tag of a list of keys fetched ahead << 32) | place in that list; the tags' top bit tells them apart
    // rows of the coming batch fetched ahead of its Read (Section 4.2), [max_ids] each: the listed keys, where a key's
    // row is staged if its write-back is still to come (else KEY_NONE: it comes from the table), and the rows
    uint32_t *pf_keys, *pf_from;
    float *pf_rows, *pf_acc;
    // (selected, not indexed: indexing kernel arguments at run time would put them in scratch memory)
    __device__ __forceinline__ float *rows_of(int b) const { return b ? rows[1] : rows[0]; }
    __device__ __forceinline__ float *acc_of(int b) const { return b ? acc[1] : acc[0]; }
    __device__ __forceinline__ uint32_t *keys_of(int b) const { return b ? keys[1] : keys[0]; }
    __device__ __forceinline__ uint32_t *cg_of(int b) const { return b ? cg[1] : cg[0]; }
};

// Everything a kernel needs to know about one cache, passed by value.
struct CacheView {
    // global table (Section 3.1): rows, optimizer state, global clock c_g
    float *W, *A;
    uint32_t *Cg;         // the clocks the kernels work on: the caller's array, or its mirror in HBM for a host-backed table
    uint32_t *Cg_host;    // host-backed table: the caller's array, written through; else null
    HostLink hl;
    uint32_t vocab;
    // cache slots
    float *rows, *acc;
    float *rows0, *acc0;  // several workers: every cached row (accumulator) as it was fetched; else null
    // Early push (table in HBM, one worker): the update that fetches a missed key's row (see apply_kernel,
    // fresh rows) writes its result to the global table as well as to the slot, and early_cc[slot] is the
    // c_c at which the two are equal.  A victim whose c_c is still that, and whose global clock is still
    // the c_s it was fetched at (nobody else pushed), is evicted without copying its row: Evict's push
    // has already travelled.  0: not equal at any c_c a row with updates can have.  nullptr: not in use.
    uint32_t *early_cc;
    int many;             // several workers write the global table: Evict pushes what was accumulated since the Fetch (Section 3.1)
    uint32_t freq_cap;    // light-weight LFU (Section 4.3): a row used this often is no longer kept track of; 0: exact policies
    uint32_t *slot_key;
    SlotMeta *meta;       // start clock, local clock, LRU stamp, LFU count: one 16-byte record per slot
    uint32_t n_slots;     // capacity + max_batch_ids
    uint32_t capacity;
    uint32_t max_ids;
    int64_t s;            // staleness bound
    // Find (Algorithm 2): the slot of every key of the table, SLOT_NONE where it is not cached.  One 4-byte load, which
    // a wave's sorted keys share lines of, in flight beside the key's global clock; one store to insert or erase.
    // With a hash table of the cached keys (buckets of 16 entries in 128 bytes) every Find was eight 16-byte loads
    // of a line no other lane wanted, every insert and erase a search: probe 13 -> 10.4 us and eviction 13 -> 10.2 us
    // at 106496 ids; a step of 3328 ids 42.9 -> 38.1 us, of 106496 ids 74.7 -> 71.3 us, of 409600 ids in bags
    // 316 -> 302 us.  4 bytes per row of the table, in HBM mostly a fraction of its clocks' and rows' own; a table that
    // leaves no room for them is searched through the hash table after all (key_hash.hpp), by a kernel before
    // the one that asks: slot_of then holds its answers by sorted position, and the index is not kept.
    int32_t *slot_of;
    uint32_t *free_list;  // free slots in ascending order (first max_ids of them)
    uint8_t *was_free;    // per slot: free when the current lookup began (its fetches may be filling it now)
    DState *ds;
    Counters *last;       // this call's counters (one of ds->call)
    Counters *next_call;  // the other one: cleared by this call for the next
    RowGeom geom;
    int adagrad;          // element-wise Adagrad: an accumulator row beside every row
    int rowwise;          // row-wise Adagrad: one accumulator per row (acc[slot], A[key]); rows of at most one piece per lane
    int by_position;      // what slot_of is indexed by (see there)
    int direct;           // no cache: rows/acc alias the global table, a key is its own slot, there are no clocks
};

constexpr int32_t SRC_BACKING = -1;   // gather reads the global row: the key was not cached (or is refetched)
constexpr int32_t SRC_ZERO = -2;      // id outside the vocabulary: the output row is zero

constexpr int PT_THREADS = 1024;                // probe tiles: 1024 sorted positions per workgroup,
constexpr int PT_WAVES = PT_THREADS / WAVE;     // one per thread, so every probe's loads are in flight at once
constexpr int PT_TILE = PT_THREADS;
constexpr int VERIFY_TILE = 1024;                    // positions one workgroup of the id check covers

// Per-call workspaces (sized by max_batch_ids unless noted).  Per-key facts are stored at the
// key's head position in the sorted order.
struct Workspace {
    uint32_t *skey, *perm;        // sorted keys and their original positions
    int32_t *src;                 // per sorted position: slot to gather from, or SRC_*
    int32_t *head_slot;           // at heads: slot of the key (set by fill for a missed key)
    uint8_t *cls;                 // at heads: HIT / STALE / MISS (lookup)
    uint32_t *tile_miss, *tile_stale, *tile_hit;     // per probe tile counts
    uint2 *miss_stage, *stale_stage;      // per probe tile: (head position, key) of its missed / stale keys
    uint32_t *bag_of;             // pooled: bag of each original position, as the lookup's offsets had it
};

// CheckValid (Section 3.1): c_c <= c_s + s and c_g <= c_c + s, as differences so that an
// "infinite" s cannot overflow.
__device__ __forceinline__ bool check_valid(uint32_t cs, uint32_t cc, uint32_t cg, int64_t s)
{
    return (int64_t)cc - (int64_t)cs <= s && (int64_t)cg - (int64_t)cc <= s;
}

__device__ __forceinline__ void count2(unsigned long long *a, unsigned long long *b, uint32_t v)
{
    if (v) { atomicAdd(a, (unsigned long long)v); atomicAdd(b, (unsigned long long)v); }
}

// ---- Evict(): policy trim ---------------------------------------------------------------------
// The victims are the m = size - capacity cached rows smallest in (last_use, slot) [LRU] or
// (freq, last_use, slot) [LFU].  A most-significant-digit radix select finds the policy key
// tau of the m-th smallest row; rows below tau go, and of the rows equal to tau the first few in
// slot order.
// The two first digits' histograms are kept from call to call (see kept_bin), so up to 4 million iterations the
// select is a look-up and one count of the rows below and at tau.
// Under LFU only rows of use count 1 can go: a trim never has more to drop than the lookup before it
// fetched (the cache was within its capacity before), and the rows that lookup fetched all have
// count 1, so the m-th smallest has count 1 too.  So the policy key is last_use under both policies,
// `key_bits` wide (last_use is at most t), and LFU's select simply passes over the rows of a higher
// count.  (With (freq, last_use) as the key a select had three passes and a kernel of its own for
// its last stage from iteration 2048 on: 11.4 us of an 87 us step at 206 000 slots.)
constexpr int SEL_BITS = 11;
constexpr int SEL_BINS = 1 << SEL_BITS;
constexpr int KEPT_BITS = 2 * SEL_BITS;                       // the policy key's top digits, counted in the kept histograms
constexpr uint32_t KEPT_WORDS = SEL_BINS + (1u << KEPT_BITS); // their words: [SEL_BINS] by the first digit, then [SEL_BINS][SEL_BINS]
constexpr int TRIM_THREADS = 256;
constexpr int TRIM_WAVES = TRIM_THREADS / WAVE;
constexpr int TRIM_ITEMS = 4;
constexpr int TRIM_TILE = TRIM_THREADS * TRIM_ITEMS;   // 1024 slots per counting tile

struct TrimPlan {
    int lfu;          // policy
    int key_bits;     // bits of the policy key (last_use): KEPT_BITS, or as many as the iteration has beyond that
    int passes;       // its digits: 2, or 3 beyond KEPT_BITS bits
    uint32_t t_now;   // iteration of the Read that left the overflow
    uint32_t *coarse, *fine;           // the kept histograms of all evictable rows, by the first digit and by both (see kept_bin)
    uint32_t *hist;                    // [SEL_BINS]: third digit, of the rows that share tau's first two
    uint32_t *zero_from;               // cleared by every Read: sup_cnt and, if there is a third digit, hist behind it
    uint32_t zero_words;
    uint4 *blk_cnt, *sup_cnt;          // per 1024 slots, and per EV_SUPER such blocks: cached rows with a policy key
                                       // below the threshold (x), equal to it (y), and those of each that hold updates (z, w)
    uint32_t *tile_free;               // free slots per 1024-slot tile
    uint32_t *ev_ids;                  // ids dropped by this trim
    int ev_slot;                       // which of the two evicted-id counts (and staging buffers) this trim appends to
    uint32_t push_seq;                 // host-backed table: serial number of this trim (never 0)
    int fetched_dirty;                 // the count ran beside the lookup's fetches, and the batch has been updated since
    uint32_t dirty_stamp;              // the count runs beside the optimizer step of the Read of this iteration's keys (0: it does not):
                                       // every row that Read touched will hold updates when the step is done, whether its clock has moved yet or not
};

__device__ __forceinline__ uint32_t policy_key(const uint4 &meta) { return meta.z; }
// Can the row be evicted at all?  (See above: under LFU only rows used once.)
__device__ __forceinline__ bool evictable(const TrimPlan &tp, const uint4 &meta) { return !tp.lfu || meta.w == 1u; }

// The kept histograms count every evictable row by the top KEPT_BITS bits of its policy key.  They need not be
// counted anew for every trim: a Read changes the keys of the rows it finds and adds the rows it fetches, a
// trim removes its victims, nothing else touches policy keys.  So the probe moves the rows it touches from
// their old bin to their new one, and the eviction takes its victims out (kept_remove_victims).  Up to iteration
// 2^22 a bin is one iteration and tau is known as soon as the probe has ended, so the rows below and at
// it are counted beside the lookup's fetches (16 MB; with the first digit's histogram kept alone, the second was
// counted beside the fetches and the rows by the update or, between two Reads, by a kernel of their own: lookups of
// 53248 ids 60.5 -> 58.4 us; and the eviction could not run beside the update, see evict_body).
// Beyond, the bins widen by a factor of two at iterations 2^22, 2^23, ...; kept_recount_kernel then counts them afresh.
// A third digit is then counted beside the fetches and the rows by the update, and the eviction has a kernel of its own: 106496
// ids 54.3 -> 58.5 us a step, 114688 ids of 128 floats 81.5 -> 86.4, 409600 ids in bags 235 -> 286, lookups of 53248 ids
// 53.6 -> 56.4, 3328 ids 36.7 -> 37.4.
__device__ __forceinline__ uint32_t kept_bin(const TrimPlan &tp, uint32_t key) { return key >> (tp.key_bits - KEPT_BITS); }

// The digit whose cumulative count first reaches `remaining`, which becomes what is left to find inside it.
// c: the counts of the thread's SEL_BINS / TRIM_THREADS consecutive digits.  Every thread gets the same answer.
constexpr int SEL_PER = SEL_BINS / TRIM_THREADS;
static_assert(SEL_PER == 8, "a thread's share of a histogram is two 16-byte loads");
__device__ __forceinline__ void sel_load(const uint32_t *hist, uint32_t (&c)[SEL_PER])
{
    const uint4 a = reinterpret_cast<const uint4 *>(hist)[2 * threadIdx.x], b = reinterpret_cast<const uint4 *>(hist)[2 * threadIdx.x + 1];
    c[0] = a.x; c[1] = a.y; c[2] = a.z; c[3] = a.w; c[4] = b.x; c[5] = b.y; c[6] = b.z; c[7] = b.w;
}
__device__ __forceinline__ uint32_t sel_pick(const uint32_t (&c)[SEL_PER], uint32_t &remaining, uint32_t *lds_pick, uint32_t *lds_scan)
{
    uint32_t s = 0, tot;
#pragma unroll
    for (int q = 0; q < SEL_PER; ++q) s += c[q];
    uint32_t run = block_excl_scan<TRIM_WAVES>(s, lds_scan, tot);
#pragma unroll
    for (int q = 0; q < SEL_PER; ++q) {
        if (c[q] && run < remaining && remaining <= run + c[q]) { lds_pick[0] = threadIdx.x * SEL_PER + q; lds_pick[1] = run; }
        run += c[q];
    }
    __syncthreads();
    const uint32_t digit = lds_pick[0] & (SEL_BINS - 1);
    remaining -= lds_pick[1];
    __syncthreads();
    return digit;
}

// Replays the select's decisions on its first `upto` digits (2 or 3): the key prefix chosen (in the high bits),
// how many of the m victims share the first digit (in_coarse) and how many the whole prefix (remaining).
// tau mostly has the present iteration's first digit, so that row of `fine` is asked for along with `coarse`.
__device__ __forceinline__ void sel_replay(const TrimPlan &tp, int upto, uint32_t m, uint32_t &prefix, uint32_t &in_coarse, uint32_t &remaining,
                                           uint32_t *lds_pick, uint32_t *lds_scan)
{
    uint32_t c[SEL_PER], f[SEL_PER];
    const uint32_t guess = kept_bin(tp, tp.t_now) >> SEL_BITS;
    sel_load(tp.coarse, c);
    sel_load(tp.fine + (size_t)guess * SEL_BINS, f);
    remaining = m;
    const uint32_t d0 = sel_pick(c, remaining, lds_pick, lds_scan);
    in_coarse = remaining;
    if (d0 != guess) sel_load(tp.fine + (size_t)d0 * SEL_BINS, f);
    const uint32_t d1 = sel_pick(f, remaining, lds_pick, lds_scan);
    prefix = (d0 << SEL_BITS | d1) << (tp.key_bits - KEPT_BITS);
    if (upto < 3) return;
    sel_load(tp.hist, c);
    prefix |= sel_pick(c, remaining, lds_pick, lds_scan);
}

// LDS of the select (a workgroup of TRIM_THREADS threads).
struct TrimLds {
    uint32_t bins[SEL_BINS];
    uint32_t pick[2];
    uint32_t scan[TRIM_WAVES + 1];
};

// Kernels that carry a stage of the next minibatch's sort give it their first workgroups (its
// chain of dependent steps is the longest, so it starts first) and number their own from
// there.  All roles of a kernel share one dynamically sized LDS buffer; the host sizes it for
// the largest role present.
extern __shared__ __align__(16) unsigned char dyn_lds[];
template <typename T> __device__ __forceinline__ T &lds_as() { return *reinterpret_cast<T *>(dyn_lds); }

// Up to two sort stages, of two different announced batches, travel in one kernel.  Returns
// true if this workgroup ran one of them; otherwise bid / nblk number the kernel's own workgroups.
__device__ __forceinline__ bool run_carried(const SortStage &a, const SortStage &b, uint32_t &bid, uint32_t &nblk)
{
    uint32_t *lds = reinterpret_cast<uint32_t *>(dyn_lds);
    if (bid < a.blocks + b.blocks) {
        const bool first = bid < a.blocks;
        sort_stage_body<SORT_THREADS>(first ? a : b, first ? bid : bid - a.blocks, lds);
        return true;
    }
    bid -= a.blocks + b.blocks; nblk -= a.blocks + b.blocks;
    return false;
}

// The third digit's histogram, over the rows whose first two are tau's.  Runs in `nblocks` workgroups of
// TRIM_THREADS threads; `vblock` is this one's index.
// It runs beside the lookup's fetches: slots that were free when the lookup began are skipped (they are being
// filled right now), and the rows fetched into them, which all carry the policy key t_now, are counted from
// their number.
__device__ __forceinline__ void trim_hist_body(const CacheView &cv, const TrimPlan &tp, const uint32_t *tile_miss, uint32_t ptiles, uint32_t vblock, uint32_t nblocks, TrimLds &l)
{
    const uint32_t new_rows = block_sum_array<TRIM_WAVES>(tile_miss, ptiles, l.scan);
    const int32_t over = cv.ds->size_before + (int32_t)new_rows - (int32_t)cv.capacity;
    if (over <= 0) return;
    uint32_t prefix, in_coarse, remaining;
    sel_replay(tp, 2, (uint32_t)over, prefix, in_coarse, remaining, l.pick, l.scan);
    for (int b = threadIdx.x; b < SEL_BINS; b += TRIM_THREADS) l.bins[b] = 0;
    __syncthreads();
    const int width = tp.key_bits - KEPT_BITS;         // 1 to 10 bits
    const uint32_t mask = (1u << width) - 1u;
    if (vblock == 0 && threadIdx.x == 0 && new_rows && (tp.t_now >> width) == (prefix >> width)) atomicAdd(&tp.hist[tp.t_now & mask], new_rows);
    for (uint32_t slot = vblock * TRIM_THREADS + threadIdx.x; slot < cv.n_slots; slot += nblocks * TRIM_THREADS) {
        const bool skip = cv.was_free[slot] != 0;
        const uint4 m = load_meta(cv.meta, slot);
        if (skip || !evictable(tp, m) || (policy_key(m) >> width) != (prefix >> width)) continue;
        atomicAdd(&l.bins[policy_key(m) & mask], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < SEL_BINS; b += TRIM_THREADS)
        if (l.bins[b]) atomicAdd(&tp.hist[b], l.bins[b]);
}

// All rows in bins below tau's were evicted, and of that bin as many as the select still had to find there.  One
// workgroup of TRIM_THREADS threads, after every other reader of the kept histograms.
__device__ __forceinline__ void kept_remove_victims(const CacheView &cv, const TrimPlan &tp, uint32_t *lds_pick, uint32_t *lds_scan)
{
    const int32_t over = cv.ds->over;
    if (over <= 0) return;
    uint32_t prefix, in_coarse, remaining;
    sel_replay(tp, 2, (uint32_t)over, prefix, in_coarse, remaining, lds_pick, lds_scan);       // (ends with a barrier: every thread has read its bins)
    const uint32_t bin = kept_bin(tp, prefix), d0 = bin >> SEL_BITS, d1 = bin & (SEL_BINS - 1);
    for (uint32_t b0 = 0; b0 < d0; b0 += TRIM_THREADS) {
        const uint32_t b = b0 + threadIdx.x;
        const uint32_t rows = b < d0 ? tp.coarse[b] : 0u;
        if (rows) tp.coarse[b] = 0;
        for (uint64_t m = __ballot(rows != 0); m; m &= m - 1) {           // (few: the rows of a first digit are evicted together once)
            uint4 *f = reinterpret_cast<uint4 *>(tp.fine + (size_t)(b - lane_id() + (uint32_t)__builtin_ctzll(m)) * SEL_BINS);
            for (uint32_t i = lane_id(); i < SEL_BINS / 4; i += WAVE) f[i] = make_uint4(0, 0, 0, 0);
        }
    }
    for (uint32_t b = threadIdx.x; b < d1; b += TRIM_THREADS) tp.fine[(size_t)d0 * SEL_BINS + b] = 0;
    if (threadIdx.x == 0) { tp.fine[bin] -= remaining; tp.coarse[d0] -= in_coarse; }
}

// The kept histograms from nothing, for the rows cached before a Read (its probe moves on from there).
static __global__ __launch_bounds__(TRIM_THREADS) void kept_recount_kernel(CacheView cv, TrimPlan tp)
{
    for (uint32_t slot = blockIdx.x * TRIM_THREADS + threadIdx.x; slot < cv.n_slots; slot += gridDim.x * TRIM_THREADS) {
        const uint4 m = load_meta(cv.meta, slot);
        if (cv.slot_key[slot] == KEY_NONE || !evictable(tp, m)) continue;
        const uint32_t bin = kept_bin(tp, policy_key(m));
        atomicAdd(&tp.fine[bin], 1u);
        atomicAdd(&tp.coarse[bin >> SEL_BITS], 1u);
    }
}

static __global__ __launch_bounds__(256) void clear_words_kernel(uint32_t *p, uint32_t words)
{
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < words; i += gridDim.x * 256u) p[i] = 0;
}

// Sums eight values per thread over the block at once (every thread gets all sums).
// `lds` needs TRIM_WAVES * 8 words.
__device__ __forceinline__ void block_sum8(uint32_t (&v)[8], uint32_t *lds)
{
    const uint32_t lane = lane_id(), w = threadIdx.x / WAVE;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = wave_sum(v[k]);
    __syncthreads();
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) lds[w * 8 + k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        uint32_t t = 0;
#pragma unroll
        for (int ww = 0; ww < TRIM_WAVES; ++ww) t += lds[ww * 8 + k];
        v[k] = t;
    }
}

// Last stage of the select: finds tau (replaying the passes) and counts, per block of EV_SLOTS
// slots (the eviction's workgroups), the cached rows whose policy key lies below tau and those
// whose key equals it, and how many of each hold updates; sup_cnt adds these up per EV_SUPER
// blocks (zero when the select starts).  With these counts the eviction places every victim by
// arithmetic alone (count at the producer, prefix at the consumer).  A workgroup of the count
// covers COUNT_SLOTS slots, a wave of it one block of EV_SLOTS (the replay is paid once per
// workgroup, so the count uses few, the eviction many).
constexpr int EV_ITEMS = 1;
constexpr int EV_SLOTS = TRIM_THREADS * EV_ITEMS;
constexpr int EV_SUPER = 32;
constexpr int COUNT_ITEMS = EV_SLOTS / WAVE;                   // consecutive slots per lane: a wave covers EV_SLOTS
constexpr int COUNT_SLOTS = TRIM_THREADS * COUNT_ITEMS;
static_assert(TRIM_TILE % EV_SLOTS == 0, "eviction workgroups do not straddle free-list tiles");
static_assert(EV_SLOTS % WAVE == 0, "a wave of the count covers one eviction block");

// The slots of a thread: keys (KEY_NONE beyond the end) and metadata.
template <int ITEMS>
__device__ __forceinline__ void load_slots(const CacheView &cv, uint32_t slot0, uint32_t (&key)[ITEMS], uint4 (&meta)[ITEMS])
{
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool in = slot0 + i < cv.n_slots;
        key[i] = in ? cv.slot_key[slot0 + i] : KEY_NONE;
        meta[i] = in ? load_meta(cv.meta, slot0 + i) : make_uint4(0, 0, 0, 0);
    }
}

// beside_fill: the count runs beside the lookup's fetches.  Slots that were free when the lookup began are being filled
// right now; those up to the last one taken hold the fetched rows, whose policy key is t_now and which hold no
// updates yet (the eviction knows if they do by then).  Rows of the batch that were found can be victims under LRU, if the
// batch has more keys than the capacity: all tied at t_now.  The stale ones among them are being refreshed right now and
// hold no updates afterwards; CheckValid says which, whatever of the refresh is seen here: it leaves c_s = c_c = c_g = max(c_g, c_c),
// so with the new c_s c_c does not exceed it, and with the old one c_c - c_s is still above the bound if either of the two conditions failed.
__device__ __forceinline__ void trim_count_body(const CacheView &cv, const TrimPlan &tp, uint32_t vblock, TrimLds &l, bool beside_fill = false,
                                                const uint32_t *tile_miss = nullptr, uint32_t ptiles = 0)
{
    uint32_t key[COUNT_ITEMS];
    uint4 meta[COUNT_ITEMS];
    const uint32_t slot0 = vblock * COUNT_SLOTS + threadIdx.x * COUNT_ITEMS;
    load_slots<COUNT_ITEMS>(cv, slot0, key, meta);      // loads first: they overlap the replay
    uint32_t last_new = 0, misses = 0;
    int32_t over;
    if (beside_fill) {
#pragma unroll
        for (int i = 0; i < COUNT_ITEMS; ++i)
            if (slot0 + i < cv.n_slots && cv.was_free[slot0 + i]) key[i] = KEY_NONE;
        misses = block_sum_array<TRIM_WAVES>(tile_miss, ptiles, l.scan);
        over = cv.ds->size_before + (int32_t)misses - (int32_t)cv.capacity;
        if (misses) last_new = cv.free_list[misses - 1];
    } else {
        over = cv.ds->size - (int32_t)cv.capacity;
    }
    if (vblock == 0 && threadIdx.x == 0) { cv.ds->over = over; cv.ds->cut_slot = -1; }
    if (over <= 0) return;
    uint32_t tau, in_coarse, take_eq;
    sel_replay(tp, tp.passes, (uint32_t)over, tau, in_coarse, take_eq, l.pick, l.scan);
    const bool new_tied = misses && tau == tp.t_now;
    uint32_t lt = 0, eq = 0, dlt = 0, deq = 0;
#pragma unroll
    for (int i = 0; i < COUNT_ITEMS; ++i) {
        const bool cached = key[i] != KEY_NONE && evictable(tp, meta[i]);
        const uint32_t pk = policy_key(meta[i]);
        bool dirty = meta[i].y > meta[i].x || (tp.dirty_stamp && meta[i].z == tp.dirty_stamp);
        if (beside_fill && dirty && cached && pk == tp.t_now && pk == tau) dirty = check_valid(meta[i].x, meta[i].y, cv.Cg[key[i]], cv.s);
        if (cached && pk < tau) { lt += 1; dlt += dirty; }
        else if (cached && pk == tau) { eq += 1; deq += dirty; }
        else if (new_tied && key[i] == KEY_NONE && slot0 + i <= last_new) eq += 1;      // (a free slot up to the last one taken)
    }
    // counts of an eviction block stay below 2^16: two to a word
    const uint32_t a = wave_sum(lt | (eq << 16));
    const uint32_t b = wave_sum(dlt | (deq << 16));
    const uint32_t eblk = vblock * TRIM_WAVES + threadIdx.x / WAVE;               // the eviction block this wave covered
    if (lane_id() == 0 && eblk * EV_SLOTS < cv.n_slots) {
        const uint4 c = make_uint4(a & 0xFFFFu, a >> 16, b & 0xFFFFu, b >> 16);
        tp.blk_cnt[eblk] = c;
        uint32_t *sup = reinterpret_cast<uint32_t *>(&tp.sup_cnt[eblk / EV_SUPER]);
        if (c.x) atomicAdd(&sup[0], c.x);
        if (c.y) atomicAdd(&sup[1], c.y);
        if (c.z) atomicAdd(&sup[2], c.z);
        if (c.w) atomicAdd(&sup[3], c.w);
    }
    if (vblock == 0 && threadIdx.x == 0) {
        cv.ds->sel_tau = tau; cv.ds->sel_take = take_eq;
        if (new_tied && take_eq) cv.ds->cut_slot = (int32_t)cv.free_list[min(take_eq, misses) - 1];     // (only fetched rows are tied: they took the first free slots in order)
    }
}

// The count where no kernel carries it.
static __global__ __launch_bounds__(TRIM_THREADS) void trim_stage_kernel(CacheView cv, TrimPlan tp)
{
    __shared__ TrimLds l;
    trim_count_body(cv, tp, blockIdx.x, l);
}

// Lists the free slots of one 1024-slot tile in ascending order behind those of the earlier
// tiles (only the first max_ids are ever needed).  tile_free holds the free count of every
// tile, left by the last trim; the idle twin of that array is cleared for the next trim.
// Workgroup of PT_THREADS threads, one slot each.
__device__ __forceinline__ void free_list_body(const CacheView &cv, const uint32_t *tile_free, uint32_t *tile_free_idle, uint32_t ev_idle,
                                               uint32_t tile, uint32_t *lds)
{
    if (threadIdx.x == 0) tile_free_idle[tile] = 0;
    if (tile == 0 && threadIdx.x == 0) cv.ds->ev_n[ev_idle] = 0;      // (push_n is written by every eviction, and a write-back on its way may still read it)
    const uint32_t slot = tile * PT_TILE + threadIdx.x;
    const bool fr = slot < cv.n_slots && cv.slot_key[slot] == KEY_NONE;
    if (slot < cv.n_slots) cv.was_free[slot] = fr ? 1 : 0;
    const uint32_t before = block_sum_array<PT_WAVES>(tile_free, tile, lds);
    if (before >= cv.max_ids) return;
    uint32_t tot;
    const uint32_t pos = before + block_excl_scan<PT_WAVES>(fr ? 1u : 0u, lds, tot);
    if (fr && pos < cv.max_ids) cv.free_list[pos] = slot;
}

// Find for every sorted position; at the head of every run of equal keys also CheckValid and
// the policy's use count.  LOOKUP: classifies HIT / STALE / MISS, stages missed and stale keys
// per tile for the fill kernel and tells the gather where each position's row comes from.
// Otherwise (update that sorted its own ids): only resolves slots and flags keys not cached.
// Compares one tile of a sorted order with the ids it was built from (PT_THREADS threads).
__device__ __forceinline__ void check_order_body(const CacheView &cv, const Workspace &ws, const int64_t *__restrict__ ids, uint32_t n, uint32_t tile)
{
    const uint32_t j = tile * PT_TILE + threadIdx.x;
    bool changed = false;
    if (j < n) {
        const int64_t id = ids[ws.perm[j]];
        const uint32_t expect = (id < 0 || id >= (int64_t)cv.vocab) ? cv.vocab : (uint32_t)id;
        changed = expect != ws.skey[j];
    }
    if (__any(changed) && lane_id() == 0) atomicOr(&cv.ds->err, ERRBIT_STATE);
}

template <bool LOOKUP>
__global__ __launch_bounds__(PT_THREADS) __attribute__((amdgpu_num_sgpr(96))) void probe_kernel(CacheView cv, Workspace ws, uint32_t n, uint32_t t_now, uint32_t ptiles,
                                                           const uint32_t *tile_free, uint32_t *tile_free_idle, uint32_t ev_idle,
                                                           TrimPlan tp,
                                                           const int64_t *__restrict__ check_ids, int pf_idle,
                                                           uint32_t *__restrict__ inv)
{
    __shared__ uint32_t lds[PT_WAVES + 1];
    // rows entering (+) and leaving (-) the kept bins: by how many bins they lie before the present one, and by the
    // first digit the same way (the present one and the one before: what lies further back goes to memory at once)
    __shared__ uint32_t kept_delta[LOOKUP ? SEL_BINS : 1], coarse_delta[2];
    const uint32_t check_blocks = LOOKUP && check_ids ? ptiles : 0u;
    if (blockIdx.x >= ptiles && blockIdx.x < ptiles + check_blocks) {
        // An order that was sorted ahead of this call (an announced batch) is checked against the ids
        // as they are now: the announcement promised they would not change.  Workgroups of their own,
        // on compute units the probe leaves idle.
        check_order_body(cv, ws, check_ids, n, blockIdx.x - ptiles);
        return;
    }
    if (blockIdx.x >= ptiles) {          // extra workgroups of a lookup: the free list for the fill kernel
        // ... and clean counts for the trim that follows this lookup
        const uint32_t first = ptiles + check_blocks;
        for (uint32_t i = (blockIdx.x - first) * PT_THREADS + threadIdx.x; i < tp.zero_words; i += (gridDim.x - first) * PT_THREADS) tp.zero_from[i] = 0;
        free_list_body(cv, tile_free, tile_free_idle, ev_idle, blockIdx.x - first, lds);
        return;
    }
    const uint32_t tile = blockIdx.x;
    const uint32_t vocab = cv.vocab;
    const uint32_t j = tile * PT_TILE + threadIdx.x;
    DState *ds = cv.ds;
    if (LOOKUP && inv && j < n) inv[ws.perm[j]] = j;         // pooled lookup: the sorted position of every original position
    const uint32_t bin_now = LOOKUP ? kept_bin(tp, t_now) : 0u;
    if (LOOKUP) {
        for (int b = threadIdx.x; b < SEL_BINS; b += PT_THREADS) kept_delta[b] = 0;
        if (threadIdx.x < 2) coarse_delta[threadIdx.x] = 0;
        __syncthreads();
    }

    if (tile == 0 && threadIdx.x == 0) {                      // this call's bookkeeping
        Counters z{};
        *cv.next_call = z;
        cv.last->n = n;
        atomicAdd(&ds->total.n, (unsigned long long)n);
        if (LOOKUP) { ds->t = t_now; ds->size_before = ds->size; }
        if (LOOKUP && pf_idle >= 0) ds->pf_n[pf_idle] = 0;    // the list of keys to fetch ahead that this lookup's second kernel may fill
    }
    // Find runs once per key, not once per position: by the head of every run of equal keys, and by
    // each wave's first lane (its run may have begun in the wave before); the other positions of a
    // run take where their row comes from from the nearest such lane below them.
    bool head = false, miss = false, stale = false, hit = false, absent = false, bad = false, finder = false, moved = false;
    int32_t my_src = SRC_ZERO;
    if (j < n) {
        const uint32_t key = ws.skey[j];
        if (key == vocab) {                                   // id outside the vocabulary
            bad = true;
            if (LOOKUP) ws.src[j] = SRC_ZERO;
            ws.head_slot[j] = SLOT_NONE;
            if (j == 0) ds->n_valid = 0;                      // not one valid id in the call
        } else {
            head = j == 0 || ws.skey[j - 1] != key;
            if (j + 1 == n || ws.skey[j + 1] == vocab) ds->n_valid = j + 1;    // one writer: the last valid position
            finder = head || (LOOKUP && lane_id() == 0);
            if (finder) {
                const uint32_t cg = LOOKUP ? cv.Cg[key] : 0u;        // in flight together with the probe's loads
                const int32_t slot = cv.slot_of[cv.by_position ? j : key];
                int32_t src = slot == SLOT_NONE ? SRC_BACKING : slot;
                bool valid = true;
                uint4 m = make_uint4(0, 0, 0, 0);
                if (LOOKUP && slot != SLOT_NONE) {
                    m = load_meta(cv.meta, (uint32_t)slot);
                    const uint32_t cs = m.x, cc = m.y;
                    valid = check_valid(cs, cc, cg, cv.s);
                    // A stale row that holds no updates of its own is refetched: its value is the
                    // global row.  (One with updates is pushed first, so its own value stays current.)
                    if (!valid && !(cc > cs)) src = SRC_BACKING;
                }
                my_src = src;
                if (head) {
                    ws.head_slot[j] = slot;
                    if (LOOKUP) {
                        if (slot == SLOT_NONE) miss = true;
                        else {
                            hit = valid; stale = !valid;
                            const bool upkeep = !(cv.freq_cap && m.w >= cv.freq_cap);        // (light-weight LFU: frequent enough, left alone)
                            if (upkeep) store_meta(cv.meta, (uint32_t)slot, m.x, m.y, t_now, m.w + 1);   // one use per key per Read
                            if (upkeep && evictable(tp, m)) {
                                const uint32_t bin_old = kept_bin(tp, policy_key(m)), back = bin_now - bin_old;
                                if (tp.lfu || back) {                    // (LFU: used twice now, out of reach)
                                    moved = !tp.lfu;
                                    if (back < (uint32_t)SEL_BINS) atomicSub(&kept_delta[back], 1u);
                                    else { atomicSub(&tp.fine[bin_old], 1u); atomicSub(&tp.coarse[bin_old >> SEL_BITS], 1u); }
                                }
                            }
                        }
                        ws.cls[j] = (uint8_t)(miss ? CLS_MISS : (stale ? CLS_STALE : CLS_HIT));
                    } else {
                        absent = slot == SLOT_NONE;
                    }
                }
            }
        }
    }
    if (LOOKUP) {
        const uint64_t below = __ballot(finder) & (~0ull >> (63u - lane_id()));
        const int from = below ? 63 - __builtin_clzll(below) : 0;
        const int32_t src = __shfl(my_src, from, WAVE);           // (a valid key has a finder at or below its lane: sorted keys, the invalid ones last)
        if (j < n && !bad) ws.src[j] = src;
    }

    if (__any(bad) && lane_id() == 0) atomicOr(&ds->err, ERRBIT_RANGE);
    if (LOOKUP) {
        const uint64_t mv = __ballot(moved);
        if (mv && lane_id() == 0) atomicAdd(&kept_delta[0], (uint32_t)__popcll(mv));
        // stage this tile's missed and stale keys, in key order, for the fill kernel
        // (a tile has 1024 positions: two counts to a word, one pass of barriers for each pair)
        uint32_t tot_ms;
        const uint32_t ms = block_excl_scan<PT_WAVES>((miss ? 1u : 0u) | (stale ? 1u << 16 : 0u), lds, tot_ms);
        const uint32_t mo = ms & 0xFFFFu, so = ms >> 16, tot_miss = tot_ms & 0xFFFFu, tot_stale = tot_ms >> 16;
        if (miss) ws.miss_stage[tile * PT_TILE + mo] = make_uint2(j, ws.skey[j]);
        if (stale) ws.stale_stage[tile * PT_TILE + so] = make_uint2(j, ws.skey[j]);
        const uint32_t tot_hit = block_sum<PT_WAVES>(hit ? 1u : 0u, lds);
        if (threadIdx.x == 0) {
            ws.tile_miss[tile] = tot_miss;
            ws.tile_stale[tile] = tot_stale;
            ws.tile_hit[tile] = tot_hit;              // (the call's counters: added up by a workgroup of the next kernel)
            if (tot_miss) atomicAdd(&kept_delta[0], tot_miss);            // the rows being fetched
        }
        __syncthreads();
        for (uint32_t b = threadIdx.x; b < (uint32_t)SEL_BINS; b += PT_THREADS) {
            const uint32_t d = kept_delta[b];
            if (d) {                                                      // (differences, modulo 2^32)
                atomicAdd(&tp.fine[bin_now - b], d);
                atomicAdd(&coarse_delta[(bin_now >> SEL_BITS) - ((bin_now - b) >> SEL_BITS)], d);
            }
        }
        __syncthreads();
        if (threadIdx.x < 2 && coarse_delta[threadIdx.x]) atomicAdd(&tp.coarse[(bin_now >> SEL_BITS) - threadIdx.x], coarse_delta[threadIdx.x]);
    } else {
        if (__any(absent) && lane_id() == 0) atomicOr(&ds->err, ERRBIT_STATE);
        const uint32_t tot_heads = block_sum<PT_WAVES>(head ? 1u : 0u, lds);
        if (threadIdx.x == 0) count2(&cv.last->unique, &ds->total.unique, tot_heads);
    }
}

// No cache (the paper's baseline "Hybrid (w/o Cache)", Section 5): Read and Write go straight to
// the global table.  The sorted order is used as it is; a key stands for its own row.
template <bool LOOKUP>
__global__ __launch_bounds__(PT_THREADS) __attribute__((amdgpu_num_sgpr(96))) void direct_probe_kernel(CacheView cv, Workspace ws, uint32_t n, uint32_t t_now, uint32_t ptiles,
                                                                  const int64_t *__restrict__ check_ids, uint32_t *__restrict__ inv)
{
    __shared__ uint32_t lds[PT_WAVES + 1];
    if (blockIdx.x >= ptiles) { check_order_body(cv, ws, check_ids, n, blockIdx.x - ptiles); return; }     // (an order sorted ahead, see probe_kernel)
    const uint32_t j = blockIdx.x * PT_TILE + threadIdx.x;
    if (LOOKUP && inv && j < n) inv[ws.perm[j]] = j;         // pooled lookup (see probe_kernel)
    const uint32_t vocab = cv.vocab;
    DState *ds = cv.ds;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        Counters z{};
        *cv.next_call = z;
        cv.last->n = n;
        atomicAdd(&ds->total.n, (unsigned long long)n);
        if (LOOKUP) ds->t = t_now;
    }
    bool head = false, bad = false;
    if (j < n) {
        const uint32_t key = ws.skey[j];
        if (key == vocab) {
            bad = true;
            if (LOOKUP) ws.src[j] = SRC_ZERO;
            ws.head_slot[j] = SLOT_NONE;
            if (j == 0) ds->n_valid = 0;
        } else {
            head = j == 0 || ws.skey[j - 1] != key;
            if (j + 1 == n || ws.skey[j + 1] == vocab) ds->n_valid = j + 1;
            if (LOOKUP) ws.src[j] = (int32_t)key;
            ws.head_slot[j] = (int32_t)key;
            if (LOOKUP && head) ws.cls[j] = (uint8_t)CLS_MISS;        // every key comes from the global table
        }
    }
    if (__any(bad) && lane_id() == 0) atomicOr(&ds->err, ERRBIT_RANGE);
    const uint32_t tot_heads = block_sum<PT_WAVES>(head ? 1u : 0u, lds);
    if (threadIdx.x == 0) count2(&cv.last->unique, &ds->total.unique, tot_heads);
}

// Evict's push for one row (Section 3.1): copy the row (and the accumulator) to the global
// table; the group's first lane sets c_g = max(c_g, c_c).  Called by a whole row group.
template <int VEC>
__device__ __forceinline__ void push_row(const CacheView &cv, uint32_t key, uint32_t slot, int gl)
{
    const RowGeom g = cv.geom;
    row_copy<VEC>(cv.W + (size_t)key * g.dim, cv.rows + (size_t)slot * g.dim, g.chunks, g.lanes, gl);
    if (cv.adagrad)
        row_copy<VEC>(cv.A + (size_t)key * g.dim, cv.acc + (size_t)slot * g.dim, g.chunks, g.lanes, gl);
    if (cv.rowwise && gl == 0) cv.A[key] = cv.acc[slot];
    if (gl == 0) {
        const uint32_t cc = cv.meta[slot].cc;
        if (cc > cv.Cg[key]) { cv.Cg[key] = cc; if (cv.Cg_host) cv.Cg_host[key] = cc; }
    }
}

// Element-wise w + (x - b): what the server holds after a worker that fetched b and now holds x has pushed.
__device__ __forceinline__ float delta_add(float w, float x, float b) { return w + (x - b); }
__device__ __forceinline__ float4 delta_add(float4 w, float4 x, float4 b)
{
    return make_float4(w.x + (x.x - b.x), w.y + (x.y - b.y), w.z + (x.z - b.z), w.w + (x.w - b.w));
}

// Several workers (Section 3.1, Evict as the paper words it): the worker pushes what it accumulated on
// the row since its Fetch and the server adds it to the global row, c_g = max(c_g, c_c).  With
// `refetch` the cached row then becomes the global row again (the Fetch that follows an Evict(key)
// in Algorithm 2; a row without updates of its own is only fetched); without, the replica keeps its
// view (flush).  Either way it counts its changes anew from here.  Called by a whole row group.
template <int VEC>
__device__ __forceinline__ void sync_row_many(const CacheView &cv, uint32_t key, uint32_t slot, int gl, bool has_updates, bool refetch)
{
    using V = typename VecT<VEC>::type;
    const RowGeom g = cv.geom;
    for (int pass = 0; pass < (cv.adagrad ? 2 : 1); ++pass) {
        V *glob = reinterpret_cast<V *>((pass ? cv.A : cv.W) + (size_t)key * g.dim);
        V *mine = reinterpret_cast<V *>((pass ? cv.acc : cv.rows) + (size_t)slot * g.dim);
        V *base = reinterpret_cast<V *>((pass ? cv.acc0 : cv.rows0) + (size_t)slot * g.dim);
        for (int c = gl; c < g.chunks; c += g.lanes) {
            V w = glob[c];
            const V x = mine[c];
            if (has_updates) { w = delta_add(w, x, base[c]); glob[c] = w; }
            if (refetch) { mine[c] = w; base[c] = w; }
            else base[c] = x;
        }
    }
    if (gl == 0 && has_updates) {
        const uint32_t cc = cv.meta[slot].cc;
        if (cc > cv.Cg[key]) cv.Cg[key] = cc;
    }
}

// Fetch's pull for one row: copy the global row (and the accumulator) into the slot.
template <int VEC>
__device__ __forceinline__ void pull_row(const CacheView &cv, uint32_t key, uint32_t slot, int gl)
{
    const RowGeom g = cv.geom;
    row_copy<VEC>(cv.rows + (size_t)slot * g.dim, cv.W + (size_t)key * g.dim, g.chunks, g.lanes, gl);
    if (cv.adagrad)
        row_copy<VEC>(cv.acc + (size_t)slot * g.dim, cv.A + (size_t)key * g.dim, g.chunks, g.lanes, gl);
    if (cv.rowwise && gl == 0) cv.acc[slot] = cv.A[key];
}

// Host-backed table: writes the rows staged by trim `buf` to the global table, with their clocks.
// Runs in `nblocks` workgroups of 256 threads; `vblock` is this one's index.
// LINK_ROWS rows per row group are on their way at a time: a transfer over the host link takes
// microseconds, and what keeps the link full is the number of rows in flight, not the number of
// workgroups (few workgroups, because a compute unit that waits for the host serves its other
// waves' memory requests behind those that wait).
constexpr int LINK_ROWS = 4;
template <int VEC>
__device__ __forceinline__ void deferred_push_body(const CacheView &cv, int buf, uint32_t vblock, uint32_t nblocks)
{
    using V = typename VecT<VEC>::type;
    const RowGeom g = cv.geom;
    const uint32_t n = cv.ds->push_n[buf];
    const uint32_t gid = (vblock * 256u + threadIdx.x) / g.lanes, ngroups = nblocks * 256u / g.lanes;
    const int gl = threadIdx.x % g.lanes;
    for (uint32_t r0 = gid * LINK_ROWS; r0 < n; r0 += ngroups * LINK_ROWS) {
        uint32_t key[LINK_ROWS], at[LINK_ROWS];
#pragma unroll
        for (int k = 0; k < LINK_ROWS; ++k) {
            at[k] = r0 + k < n ? r0 + k : r0;
            key[k] = cv.hl.keys_of(buf)[at[k]];
            if (r0 + k >= n) key[k] = KEY_NONE;          // (KEY_NONE within the list: a tied victim without updates)
        }
        for (int pass = 0; pass < (cv.adagrad ? 2 : 1); ++pass) {
            const float *from = pass ? cv.hl.acc_of(buf) : cv.hl.rows_of(buf);
            float *to = pass ? cv.A : cv.W;
            static_assert(LINK_ROWS == 4, "the copy below is written out for four rows");
            for (int c = gl; c < g.chunks; c += g.lanes) {
                // (named values, not an array: with an array the compiler kept the rows in scratch
                // memory and waited for each store to the host before the next)
                const V v0 = reinterpret_cast<const V *>(from + (size_t)at[0] * g.dim)[c];
                const V v1 = reinterpret_cast<const V *>(from + (size_t)at[1] * g.dim)[c];
                const V v2 = reinterpret_cast<const V *>(from + (size_t)at[2] * g.dim)[c];
                const V v3 = reinterpret_cast<const V *>(from + (size_t)at[3] * g.dim)[c];
                if (key[0] != KEY_NONE) reinterpret_cast<V *>(to + (size_t)key[0] * g.dim)[c] = v0;
                if (key[1] != KEY_NONE) reinterpret_cast<V *>(to + (size_t)key[1] * g.dim)[c] = v1;
                if (key[2] != KEY_NONE) reinterpret_cast<V *>(to + (size_t)key[2] * g.dim)[c] = v2;
                if (key[3] != KEY_NONE) reinterpret_cast<V *>(to + (size_t)key[3] * g.dim)[c] = v3;
            }
        }
        if (gl == 0) {
#pragma unroll
            for (int k = 0; k < LINK_ROWS; ++k)
                if (key[k] != KEY_NONE) cv.Cg_host[key[k]] = cv.hl.cg_of(buf)[at[k]];
        }
    }
}

template <int VEC>
__global__ __launch_bounds__(256) void deferred_push_kernel(CacheView cv, int buf)
{
    deferred_push_body<VEC>(cv, buf, blockIdx.x, gridDim.x);
}

// Exclusive prefix of per-tile counts into LDS (ntiles <= capacity of `pre`), total returned.
template <int NW>
__device__ __forceinline__ uint32_t tile_prefix_to_lds(const uint32_t *counts, uint32_t ntiles, uint32_t *pre, uint32_t *scan)
{
    uint32_t carry = 0;
    for (uint32_t b = 0; b < ntiles; b += NW * WAVE) {
        const uint32_t i = b + threadIdx.x;
        const uint32_t v = i < ntiles ? counts[i] : 0u;
        uint32_t tot;
        const uint32_t e = block_excl_scan<NW>(v, scan, tot);
        if (i < ntiles) pre[i] = carry + e;
        carry += tot;
    }
    __syncthreads();
    return carry;
}

// Largest t with pre[t] <= m (pre ascending, pre[0] = 0).
__device__ __forceinline__ uint32_t tile_of(const uint32_t *pre, uint32_t ntiles, uint32_t m)
{
    uint32_t lo = 0, hi = ntiles;
    while (hi - lo > 1) { const uint32_t mid = (lo + hi) >> 1; if (pre[mid] <= m) lo = mid; else hi = mid; }
    return lo;
}

constexpr int MAX_PROBE_TILES = 1024;     // max_batch_ids <= 2^20 per call

// Fetch of the missed keys, Evict + Fetch of the stale ones (Algorithm 2), and Get, one row
// group per item.  The i-th missed key in ascending key order takes the i-th free slot in
// ascending slot order.  The gather reads a missed key's row from the global table (the same
// values the fetch copies), so it does not wait for the fetch: the first `fill_blocks`
// workgroups fetch, the others gather, side by side.
// POOLED: out[b] = sum of the bag's rows in bag order; else out[perm[j]] = row of position j.
constexpr int GATHER_ROWS = 8;
constexpr int POOL_ROWS = 8;
constexpr int FILL_ROWS = 2;              // missed keys a row group fetches at a time
// A row chunk as the compiler's own vector type (arrays of these stay in registers where arrays
// of the HIP struct type of the same size did not).
typedef float raw_float4 __attribute__((ext_vector_type(4)));
template <int VEC> struct RawVecT { using type = float; };
template <> struct RawVecT<4> { using type = raw_float4; };

// Optional time stamps inside the two heavy kernels, one record of TRACE_WORDS words per workgroup
// (het_profile_trace): [0] start, [5] the last wave's end, [6] role.
// apply_kernel: roles 1 carried sort stage, 2 eviction or the count before it, 3 id check, 4 tile of the update; for
// role 4 also [1] tile and segments listed, [2] short segments done, [3] long segments done,
// [4] past the barrier before the border runs.
// fill_gather_kernel: roles 1 carried sort stage, 2 fetch, 3 the fetched keys' bookkeeping,
// 4 count of the rows to evict, 5 gather, 6 host link (write-back, list of rows to fetch ahead).
// Clock: wall_clock64(), 100 MHz.
constexpr int TRACE_WORDS = 8;
struct KernelTrace {
    unsigned long long *rec;     // nullptr: off
    uint32_t cap;                // workgroups the buffer has room for
    __device__ __forceinline__ void stamp(int i) const { if (rec && threadIdx.x == 0 && blockIdx.x < cap) rec[(size_t)blockIdx.x * TRACE_WORDS + i] = wall_clock64(); }
    __device__ __forceinline__ void end() const { if (rec && lane_id() == 0 && blockIdx.x < cap) atomicMax(&rec[(size_t)blockIdx.x * TRACE_WORDS + 5], (unsigned long long)wall_clock64()); }   // (the last wave to leave)
    __device__ __forceinline__ void role(int r) const { if (rec && threadIdx.x == 0 && blockIdx.x < cap) rec[(size_t)blockIdx.x * TRACE_WORDS + 6] = (unsigned long long)r; }
};

// Fetch's pull for FILL_ROWS rows at once (all loads first).  Called by a whole row group.
template <int VEC, bool WITH_ACC>
__device__ __forceinline__ void fetch_rows(const CacheView &cv, const float *const (&srow)[FILL_ROWS], const float *const (&sacc)[FILL_ROWS],
                                           const uint32_t (&slot)[FILL_ROWS], int nin, int gl)
{
    using V = typename RawVecT<VEC>::type;
    const RowGeom g = cv.geom;
    for (int c = gl; c < g.chunks; c += g.lanes) {
        V v[FILL_ROWS], a[FILL_ROWS];
#pragma unroll
        for (int r = 0; r < FILL_ROWS; ++r) {
            v[r] = reinterpret_cast<const V *>(srow[r])[c];
            if constexpr (WITH_ACC) a[r] = reinterpret_cast<const V *>(sacc[r])[c];
        }
#pragma unroll
        for (int r = 0; r < FILL_ROWS; ++r) {
            if (r < nin) {
                reinterpret_cast<V *>(cv.rows + (size_t)slot[r] * g.dim)[c] = v[r];
                if constexpr (WITH_ACC) reinterpret_cast<V *>(cv.acc + (size_t)slot[r] * g.dim)[c] = a[r];
                if (cv.many) {                       // several workers: the row as fetched
                    reinterpret_cast<V *>(cv.rows0 + (size_t)slot[r] * g.dim)[c] = v[r];
                    if constexpr (WITH_ACC) reinterpret_cast<V *>(cv.acc0 + (size_t)slot[r] * g.dim)[c] = a[r];
                }
            }
        }
    }
}

// Host-backed table: the rows the next Read will miss are fetched while the Write in between runs
// (Section 4.2: the next minibatch's indices are known in advance; Section 4.1: communication is
// invoked asynchronously and overlaps computation).  The second kernel of a lookup lists the keys of
// the announced batch that are not cached (nothing is inserted before that batch's own lookup, and a
// key evicted in between is found through `pend`); a kernel on a stream of its own then brings their
// rows from the table into HBM, beside the last trim's write-back going the other way; the next
// lookup's fetch kernel takes them from there.
struct Ahead {
    const uint32_t *skey;   // the announced batch's sorted keys (listing role), or null
    uint32_t n;             // their number
    uint32_t blocks;        // workgroups of the listing role in this launch
    uint32_t list_tag;      // tag the listing role gives the keys it lists (top bit set)
    int list_slot;          // which of ds->pf_n counts them
    uint32_t pending_seq;   // serial number of the trim whose staged rows are still to be written back (0: none)
    uint32_t use_tag;       // fetch role: tag of the rows that were fetched ahead for THIS lookup (0: none)
};

// Lists the keys of an announced batch that are not cached.  Workgroups of 256 threads, one sorted position each.
__device__ __forceinline__ void ahead_list_body(const CacheView &cv, const Ahead &ah, uint32_t vblock)
{
    const uint32_t j = vblock * 256u + threadIdx.x;
    bool want = false;
    uint32_t key = KEY_NONE, from = KEY_NONE;
    if (j < ah.n) {
        key = ah.skey[j];
        const bool head = key != cv.vocab && (j == 0 || ah.skey[j - 1] != key);
        if (head && cv.slot_of[cv.by_position ? j : key] == SLOT_NONE) {
            want = true;
            // a row the last trim evicted, whose write-back is still to come: the staged copy is the row
            const uint64_t pe = cv.hl.pend[key];
            if (ah.pending_seq && (uint32_t)(pe >> 32) == ah.pending_seq) from = (uint32_t)pe;
        }
    }
    const uint64_t m = __ballot(want);
    if (!m) return;
    uint32_t base = 0;
    const uint32_t first = (uint32_t)__builtin_ctzll(m);
    if (lane_id() == first) base = atomicAdd(&cv.ds->pf_n[ah.list_slot], (uint32_t)__popcll(m));     // (the order of the list does not matter)
    base = __shfl(base, (int)first, WAVE);
    if (want) {
        const uint32_t at = base + mask_rank(m);
        cv.hl.pf_keys[at] = key;
        cv.hl.pf_from[at] = from;
        cv.hl.pend[key] = ((uint64_t)ah.list_tag << 32) | at;
    }
}

// On the stream beside the main one: the first push_blocks workgroups write the rows a trim staged
// back to the table (push_buf < 0: nothing to write), the others bring the listed rows in.
template <int VEC>
__global__ __launch_bounds__(256) void link_kernel(CacheView cv, int push_buf, int list_slot, int staged_buf, uint32_t push_blocks)
{
    if (blockIdx.x < push_blocks) { if (push_buf >= 0) deferred_push_body<VEC>(cv, push_buf, blockIdx.x, push_blocks); return; }
    if (list_slot < 0) return;
    const RowGeom g = cv.geom;
    const uint32_t n = cv.ds->pf_n[list_slot];
    const uint32_t gid = ((blockIdx.x - push_blocks) * 256u + threadIdx.x) / g.lanes, ngroups = (gridDim.x - push_blocks) * 256u / g.lanes;
    const int gl = threadIdx.x % g.lanes;
    using V = typename VecT<VEC>::type;
    for (uint32_t r0 = gid * LINK_ROWS; r0 < n; r0 += ngroups * LINK_ROWS) {
        uint32_t at[LINK_ROWS], key[LINK_ROWS], from[LINK_ROWS];
#pragma unroll
        for (int k = 0; k < LINK_ROWS; ++k) {
            at[k] = r0 + k < n ? r0 + k : r0;            // (past the end: the first row again, to the same place)
            key[k] = cv.hl.pf_keys[at[k]]; from[k] = cv.hl.pf_from[at[k]];
        }
        for (int pass = 0; pass < (cv.adagrad ? 2 : 1); ++pass) {
            const float *table = pass ? cv.A : cv.W, *stage = pass ? cv.hl.acc_of(staged_buf) : cv.hl.rows_of(staged_buf);
            float *to = pass ? cv.hl.pf_acc : cv.hl.pf_rows;
            for (int c = gl; c < g.chunks; c += g.lanes) {
                V v[LINK_ROWS];
#pragma unroll
                for (int k = 0; k < LINK_ROWS; ++k) {
                    const float *row = from[k] != KEY_NONE ? stage + (size_t)from[k] * g.dim : table + (size_t)key[k] * g.dim;
                    v[k] = reinterpret_cast<const V *>(row)[c];
                }
#pragma unroll
                for (int k = 0; k < LINK_ROWS; ++k) reinterpret_cast<V *>(to + (size_t)at[k] * g.dim)[c] = v[k];
            }
        }
    }
}

// Get for bags (sum pooling): `split` row groups of a workgroup add up a bag, a contiguous share each, in bag order, in fp64;
// the shares are added in a fixed order and rounded once (a bag may hold hundreds of rows).  Where the rows are is found
// for as many ids of the share as the group has lanes at once, one id per lane (its sorted position, then source and key there:
// two steps for the whole stretch, not two per POOL_ROWS rows), and handed from lane to lane
// for the row loads; the next stretch is asked for behind the first rows of the present one.
// A row's address carries "does not count" (an id outside the vocabulary) in its lowest bit.
// split: see pool_split in the host code.
template <int VEC>
__device__ __forceinline__ void pooled_gather_body(const CacheView &cv, const Workspace &ws, uint32_t n, float *__restrict__ out,
                                                   const int64_t *__restrict__ offsets, uint32_t n_bags, const uint32_t *__restrict__ inv,
                                                   uint32_t split, uint32_t blk, uint32_t nblk_)
{
    using V = typename VecT<VEC>::type;
    const RowGeom g = cv.geom;
    const int gl = threadIdx.x % g.lanes;
    const int first_lane = (int)(threadIdx.x % WAVE) - gl;
    const uint32_t group = threadIdx.x / g.lanes, part = group % split, bags = 256u / g.lanes / split;         // bags a workgroup has in hand
    const uint32_t wave = threadIdx.x / WAVE, bag_waves = split * g.lanes / WAVE;                             // (0 or 1: a bag's groups share a wave)
    double *wave_sums = reinterpret_cast<double *>(dyn_lds);               // [waves][lanes of a row][VEC]
    auto where = [&](uint32_t jj, bool in) -> unsigned long long {
        const int32_t sr = ws.src[jj];
        const uint32_t ky = ws.skey[jj];
        const float *row = sr == SRC_BACKING ? cv.W + (size_t)ky * g.dim : cv.rows + (size_t)(uint32_t)(sr < 0 ? 0 : sr) * g.dim;
        return (unsigned long long)(uintptr_t)row | (in && sr != SRC_ZERO ? 0ull : 1ull);
    };
    for (uint32_t b0 = blk * bags; b0 < n_bags; b0 += nblk_ * bags) {
        const uint32_t b = b0 + group / split;
        int64_t lo = 0, hi = 0;
        if (b < n_bags) {
            lo = offsets[b]; hi = offsets[b + 1];
            lo = lo < 0 ? 0 : lo; hi = hi > (int64_t)n ? (int64_t)n : hi;
            if (split > 1 && lo < hi) {
                const int64_t share = (hi - lo + split - 1) / split;
                lo += part * share;
                hi = lo + share < hi ? lo + share : hi;
            }
        }
        for (int c0 = 0; c0 < g.chunks; c0 += g.lanes) {
            const bool mine = c0 + gl < g.chunks;
            const int c = mine ? c0 + gl : 0;    // (a lane beyond the row reads its first piece and stores nothing: every lane hands addresses on)
            double sum[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) sum[e] = 0.0;
            if (lo < hi) {
                int64_t i0 = lo;
                unsigned long long cur = where(inv[i0 + gl < hi ? i0 + gl : hi - 1], i0 + gl < hi);
                if (c0 == 0) for (int64_t i = lo + gl; i < hi; i += g.lanes) ws.bag_of[i] = b;
                while (i0 < hi) {
                    const int cnt = hi - i0 < (int64_t)g.lanes ? (int)(hi - i0) : g.lanes;
                    const int64_t i1 = i0 + g.lanes;
                    const bool more = i1 < hi;
                    const uint32_t jj1 = more ? inv[i1 + gl < hi ? i1 + gl : hi - 1] : 0u;
                    unsigned long long nxt = 0ull;
                    for (int r0 = 0; r0 < cnt; r0 += POOL_ROWS) {
                        V v[POOL_ROWS];
                        bool counts[POOL_ROWS];
#pragma unroll
                        for (int r = 0; r < POOL_ROWS; ++r) {
                            const int rr = r0 + r < cnt ? r0 + r : cnt - 1;
                            const unsigned long long p = __shfl(cur, first_lane + rr, WAVE);
                            counts[r] = r0 + r < cnt && !(p & 1ull);
                            v[r] = reinterpret_cast<const V *>((uintptr_t)(p & ~1ull))[c];
                        }
                        if (r0 == 0 && more) nxt = where(jj1, i1 + gl < hi);
#pragma unroll
                        for (int r = 0; r < POOL_ROWS; ++r) {
                            const float *vf = reinterpret_cast<const float *>(&v[r]);
#pragma unroll
                            for (int e = 0; e < VEC; ++e) sum[e] += counts[r] ? (double)vf[e] : 0.0;
                        }
                    }
                    cur = nxt; i0 = i1;
                }
            }
            // the shares: within the wave, then wave by wave
            for (uint32_t o = g.lanes; o < min(split * g.lanes, (uint32_t)WAVE); o <<= 1) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) sum[e] += __shfl_xor(sum[e], (int)o, WAVE);
            }
            if (bag_waves > 1) {
                __syncthreads();                 // (the sums before have been read)
                if (first_lane == 0) {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) wave_sums[(wave * g.lanes + gl) * VEC + e] = sum[e];
                }
                __syncthreads();
                if (part == 0) {
                    for (uint32_t ww = 1; ww < bag_waves; ++ww)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) sum[e] += wave_sums[((wave + ww) * g.lanes + gl) * VEC + e];
                }
            }
            V res;
            float *rf = reinterpret_cast<float *>(&res);
#pragma unroll
            for (int e = 0; e < VEC; ++e) rf[e] = (float)sum[e];
            if (mine && part == 0 && b < n_bags) reinterpret_cast<V *>(out + (size_t)b * g.dim)[c] = res;
        }
    }
}

struct FillLds {                             // (also what the pooled gather's workgroups have: a double per thread and float of a piece)
    uint32_t pre_miss[MAX_PROBE_TILES], pre_stale[MAX_PROBE_TILES];
    uint32_t scan[4 + 1];
};
static_assert(sizeof(FillLds) >= 256 * 4 * sizeof(double), "");
// RIDE: carries sort stages of announced batches.
// TRACE: time stamps (het_profile_trace); a kernel of its own, because the stamps' arguments cost the
// other one scalar registers it has no room for.
template <int VEC, bool POOLED, bool RIDE, bool TRACE>
__global__ __launch_bounds__(256) void fill_gather_kernel(CacheView cv, Workspace ws, uint32_t n, uint32_t t_now, uint32_t ptiles, uint32_t fill_blocks,
                                                          TrimPlan tp, uint32_t hist_blocks, float *__restrict__ out, const int64_t *__restrict__ offsets, uint32_t n_bags,
                                                          const uint32_t *__restrict__ inv, SortStage ride, SortStage ride2,
                                                          uint32_t push_blocks, int push_buf, uint32_t push_seq, Ahead ah,
                                                          KernelTrace tr_arg, int fetch_mode, uint32_t pool_split)
{
    using V = typename VecT<VEC>::type;
    uint32_t bid = blockIdx.x, nblk = gridDim.x;
    const KernelTrace tr = TRACE ? tr_arg : KernelTrace{nullptr, 0u};
    tr.stamp(0);
    if (RIDE && run_carried(ride, ride2, bid, nblk)) { tr.role(1); tr.end(); return; }
    if (bid < push_blocks) { deferred_push_body<VEC>(cv, push_buf, bid, push_blocks); tr.role(6); tr.end(); return; }    // host-backed table: the last trim's write-back
    bid -= push_blocks; nblk -= push_blocks;
    if (bid < ah.blocks) { ahead_list_body(cv, ah, bid); tr.role(6); tr.end(); return; }                                 // host-backed table: what to fetch ahead for the coming batch
    bid -= ah.blocks; nblk -= ah.blocks;
    const RowGeom g = cv.geom;
    const int gl = threadIdx.x % g.lanes;
    const uint32_t groups_per_block = 256u / g.lanes;
    if (POOLED) {
        // Get for bags.  These workgroups live longest (a row group adds up a whole bag), so they take
        // the first places; all the other roles' workgroups follow.
        const uint32_t others = fill_blocks + (fill_blocks && fetch_mode != 2 ? ptiles : 0u) + hist_blocks;
        const uint32_t bag_blocks = nblk - others;
        if (bid < bag_blocks) {
            if (fill_blocks == 0 && bid == 0 && threadIdx.x == 0) cv.ds->n_unique = (uint32_t)cv.last->unique;   // (no fetch workgroup does)
            pooled_gather_body<VEC>(cv, ws, n, out, offsets, n_bags, inv, pool_split, bid, bag_blocks);
            tr.role(5); tr.end();
            return;
        }
        bid -= bag_blocks; nblk -= bag_blocks;
    }
    // fetch_mode 0: everything.  1: the missed keys' rows are left to the update that follows (it reads
    // them from the global table and writes them to their slots with its step applied: they are
    // neither written nor read once more); all else as usual.  2: only those rows (a call came
    // between that is not that update).
    const uint32_t ins_blocks = fill_blocks && fetch_mode != 2 ? ptiles : 0u;
    if (bid < fill_blocks) {
        FillLds &fl = lds_as<FillLds>();
        const uint32_t tot_miss = tile_prefix_to_lds<4>(ws.tile_miss, ptiles, fl.pre_miss, fl.scan);
        const uint32_t tot_stale = tile_prefix_to_lds<4>(ws.tile_stale, ptiles, fl.pre_stale, fl.scan);
        const uint32_t gid = bid * groups_per_block + threadIdx.x / g.lanes;
        const uint32_t ngroups = fill_blocks * groups_per_block;
        if (bid == 0 && fetch_mode != 2 && threadIdx.x < WAVE) {
            // The lookup's counters, by one wave.  (Added up with atomics by every workgroup of the probe, a hundred and more
            // to one cache line, they were the last thing the probe waited for: 106496 ids 60.2 -> 58.3 us a step, 409600
            // ids in bags 251 -> 237, lookups of 53248 ids 58.5 -> 57.5.)
            uint32_t hits = 0;
            for (uint32_t i = threadIdx.x; i < ptiles; i += WAVE) hits += ws.tile_hit[i];
            hits = wave_sum(hits);
            if (threadIdx.x == 0) {
                DState *ds = cv.ds;
                const uint32_t unique = hits + tot_stale + tot_miss;
                cv.last->hit = hits; cv.last->stale = tot_stale; cv.last->miss = tot_miss; cv.last->unique = unique;
                ds->total.hit += hits; ds->total.stale += tot_stale; ds->total.miss += tot_miss; ds->total.unique += unique;
                ds->size = ds->size_before + (int32_t)tot_miss;
                ds->n_unique = unique;               // for an update that reuses this order
            }
        }
        // Fetch(k) into a new slot, FILL_ROWS keys per row group at a time: where each row comes from
        // and goes to is asked for all of them first, then the rows (few workgroups with several
        // rows in flight each leave the chip to the other roles of this kernel from the start)
        for (uint32_t m0 = gid; m0 < tot_miss && fetch_mode != 1; m0 += ngroups * FILL_ROWS) {
            const float *srow[FILL_ROWS], *sacc[FILL_ROWS];
            uint32_t slot[FILL_ROWS], keyr[FILL_ROWS];
#pragma unroll
            for (int r = 0; r < FILL_ROWS; ++r) {
                const uint32_t m = m0 + r * ngroups < tot_miss ? m0 + r * ngroups : m0;     // (beyond the end: the first row again, not stored)
                const uint32_t tl = tile_of(fl.pre_miss, ptiles, m);
                const uint32_t key = ws.miss_stage[tl * PT_TILE + (m - fl.pre_miss[tl])].y;
                keyr[r] = key;
                slot[r] = cv.free_list[m];
                // host-backed table: a row the last trim evicted may still be on its way to the table
                // (its write-back travels in this very kernel); then the staged copy is the global row
                // or it was fetched ahead into HBM for this very lookup
                const bool link = cv.Cg_host && (push_seq || ah.use_tag);
                const uint64_t pe = link ? cv.hl.pend[key] : 0ull;
                const uint32_t tag = (uint32_t)(pe >> 32);
                const bool staged = link && push_seq && tag == push_seq;
                const bool ahead = link && ah.use_tag && tag == ah.use_tag;
                const size_t at = (size_t)(uint32_t)pe * g.dim;
                srow[r] = staged ? cv.hl.rows_of(push_buf) + at : (ahead ? cv.hl.pf_rows + at : cv.W + (size_t)key * g.dim);
                sacc[r] = staged ? cv.hl.acc_of(push_buf) + at : (ahead ? cv.hl.pf_acc + at : cv.A + (size_t)key * g.dim);
            }
            int nin = 0;                         // rows of this batch that exist (the first ones)
#pragma unroll
            for (int r = 0; r < FILL_ROWS; ++r) nin += m0 + r * ngroups < tot_miss ? 1 : 0;
            if (cv.adagrad) fetch_rows<VEC, true>(cv, srow, sacc, slot, nin, gl);
            else fetch_rows<VEC, false>(cv, srow, sacc, slot, nin, gl);
            if (fetch_mode == 2 && cv.early_cc && gl == 0) {        // the update that would have pushed early is not coming
#pragma unroll
                for (int r = 0; r < FILL_ROWS; ++r)
                    if (r < nin) cv.early_cc[slot[r]] = 0u;
            }
            if (cv.rowwise && gl == 0) {             // (one accumulator per row; such a table is in HBM)
#pragma unroll
                for (int r = 0; r < FILL_ROWS; ++r)
                    if (r < nin) cv.acc[slot[r]] = cv.A[keyr[r]];
            }
        }                                        // (clocks, key and index entry: the workgroups below)
        for (uint32_t m = gid; m < tot_stale && fetch_mode != 2; m += ngroups) {                // Evict(k); Fetch(k) in place
            const uint32_t tl = tile_of(fl.pre_stale, ptiles, m);
            const uint2 jk = ws.stale_stage[tl * PT_TILE + (m - fl.pre_stale[tl])];
            const uint32_t key = jk.y;
            const uint32_t slot = (uint32_t)ws.head_slot[jk.x];
            const bool has_updates = cv.meta[slot].cc > cv.meta[slot].cs;
            if (cv.many) sync_row_many<VEC>(cv, key, slot, gl, has_updates, true);
            else if (has_updates) push_row<VEC>(cv, key, slot, gl);          // now the global row equals the cached one
            else pull_row<VEC>(cv, key, slot, gl);
            if (gl == 0) {
                const uint32_t cg = cv.Cg[key];
                cv.meta[slot].cs = cg; cv.meta[slot].cc = cg;
                if (has_updates) count2(&cv.last->stale_dirty, &cv.ds->total.stale_dirty, 1u);
                if (cv.Cg_host && !has_updates) for (uint32_t jj = jk.x; jj < n && ws.skey[jj] == key; ++jj) ws.src[jj] = (int32_t)slot;
            }
        }
        tr.role(2); tr.end();
        return;
    }

    // Fetch's bookkeeping, one thread per missed key and one workgroup per probe tile, beside the row
    // copies above (done by the same lanes it would stand behind them: two more dependent steps)
    if (bid < fill_blocks + ins_blocks) {
        const uint32_t tl = bid - fill_blocks;
        constexpr int KEYS = PT_TILE / 256;
        const uint32_t here = ws.tile_miss[tl];
        uint2 jks[KEYS];                         // (they and the clocks are on their way while the tiles before are added up)
        uint32_t cgs[KEYS];
#pragma unroll
        for (int i = 0; i < KEYS; ++i) {
            const uint32_t ml = threadIdx.x + 256u * i;
            jks[i] = ml < here ? ws.miss_stage[tl * PT_TILE + ml] : make_uint2(0, 0);
        }
#pragma unroll
        for (int i = 0; i < KEYS; ++i) cgs[i] = threadIdx.x + 256u * i < here ? cv.Cg[jks[i].y] : 0u;
        const uint32_t before = block_sum_array<4>(ws.tile_miss, tl, lds_as<FillLds>().scan);
#pragma unroll
        for (int i = 0; i < KEYS; ++i) {
            const uint32_t ml = threadIdx.x + 256u * i;
            if (ml >= here) continue;
            const uint32_t slot = cv.free_list[before + ml];
            const uint32_t j = jks[i].x, key = jks[i].y, cg = cgs[i];
            store_meta(cv.meta, slot, cg, cg, t_now, 1u);                    // c_s = c_c = c_g; first use
            if (cv.early_cc) cv.early_cc[slot] = fetch_mode == 1 ? cg + 1u : 0u;    // (the update that fetches the row will make it c_g + 1)
            cv.slot_key[slot] = key;
            ws.head_slot[j] = (int32_t)slot;
            if (!cv.by_position) cv.slot_of[key] = (int32_t)slot;
            // host-backed table: the gather runs after this kernel and reads the cached copy
            if (cv.Cg_host) for (uint32_t jj = j; jj < n && ws.skey[jj] == key; ++jj) ws.src[jj] = (int32_t)slot;
        }
        tr.role(3); tr.end();
        return;
    }
    bid -= ins_blocks; nblk -= ins_blocks;
    if (bid < fill_blocks + hist_blocks) {
        // the coming trim's select, over the rows cached before this lookup plus the rows being fetched right now
        // (known by their number and slots, not read): the count or, where there is a third digit, its histogram
        if (tp.passes == 2) trim_count_body(cv, tp, bid - fill_blocks, lds_as<TrimLds>(), true, ws.tile_miss, ptiles);
        else trim_hist_body(cv, tp, ws.tile_miss, ptiles, bid - fill_blocks, hist_blocks, lds_as<TrimLds>());
        tr.role(4); tr.end();
        return;
    }
    if (POOLED) return;                  // (never reached: the bags' workgroups came first)
    const uint32_t first_gather = fill_blocks + hist_blocks;
    if (fill_blocks == 0 && bid == 0 && threadIdx.x == 0) cv.ds->n_unique = (uint32_t)cv.last->unique;   // (no fetch workgroup did)
    const uint32_t gid = (bid - first_gather) * groups_per_block + threadIdx.x / g.lanes;
    const uint32_t ngroups = (nblk - first_gather) * groups_per_block;
    {
        // Get, GATHER_ROWS positions per row group at a time: where each row comes from is asked
        // for all of them first, then the rows themselves, so that a group has several rows in
        // flight (one row per group at a time leaves the memory system idle most of the time)
        for (uint32_t j0 = gid * GATHER_ROWS; j0 < n; j0 += ngroups * GATHER_ROWS) {
            int32_t sr[GATHER_ROWS];
            uint32_t pm[GATHER_ROWS], ky[GATHER_ROWS];
#pragma unroll
            for (int r = 0; r < GATHER_ROWS; ++r) {
                const uint32_t j = j0 + r;
                const bool in = j < n;
                sr[r] = in ? ws.src[j] : SRC_ZERO;
                pm[r] = in ? ws.perm[j] : 0u;
                ky[r] = in ? ws.skey[j] : 0u;
            }
            const float *row[GATHER_ROWS];
#pragma unroll
            for (int r = 0; r < GATHER_ROWS; ++r)     // (an id outside the vocabulary reads some row and drops it: no branch between the loads)
                row[r] = sr[r] == SRC_BACKING ? cv.W + (size_t)ky[r] * g.dim : cv.rows + (size_t)(uint32_t)(sr[r] < 0 ? 0 : sr[r]) * g.dim;
            for (int c = gl; c < g.chunks; c += g.lanes) {
                V v[GATHER_ROWS];
#pragma unroll
                for (int r = 0; r < GATHER_ROWS; ++r) v[r] = reinterpret_cast<const V *>(row[r])[c];
#pragma unroll
                for (int r = 0; r < GATHER_ROWS; ++r) {
                    if (sr[r] == SRC_ZERO) v[r] = V{};
                    if (j0 + r < n) reinterpret_cast<V *>(out + (size_t)pm[r] * g.dim)[c] = v[r];
                }
            }
        }
    }
    tr.role(5); tr.end();
}

// Pooled update: the bag of an original position (its gradient row), the last that begins at or before it.  The lookup has
// left a guess, which holds as long as the offsets are the lookup's; else it is searched for.  (A kernel of its own that searched for every
// position's bag took 4 to 5 us.)
__device__ __forceinline__ uint32_t bag_of_position(const uint32_t *bag_of, const int64_t *offsets, uint32_t n_bags, uint32_t i)
{
    const uint32_t guess = min(bag_of[i], n_bags - 1);
    const int64_t from = offsets[guess], to = offsets[guess + 1];
    if ((guess == 0 || from <= (int64_t)i) && (guess + 1 == n_bags || (int64_t)i < to)) return guess;
    uint32_t lo = 0, hi = n_bags;            // largest b with offsets[b] <= i
    while (hi - lo > 1) { const uint32_t mid = (lo + hi) / 2; if (offsets[mid] <= (int64_t)i) lo = mid; else hi = mid; }
    return lo;
}

// Hardware square root and reciprocal (about one unit in the last place each): the Adagrad
// step lr * G / (sqrt(a) + eps) tolerates that a hundred times over, and the correctly rounded
// sequences cost more instructions than everything else in the kernel.
__device__ __forceinline__ float fast_sqrt(float v) { return __builtin_amdgcn_sqrtf(v); }
__device__ __forceinline__ float fast_rcp(float v) { return __builtin_amdgcn_rcpf(v); }

// x - step, the step rounded by itself in every variant of the kernel (no fused multiply-add): a row's value does not
// depend on which of them it went through.
__device__ __forceinline__ float minus(float x, float step)
{
#pragma clang fp contract(off)
    return x - step;
}

// The optimizer of an update's kernel: known to it where rows have one piece per lane (registers), asked for beyond.
constexpr int AO_SGD = 0, AO_ADAGRAD = 1, AO_ROWWISE = 2, AO_ANY = 3;
template <int OPT> __device__ __forceinline__ bool by_adagrad(const CacheView &cv) { return OPT == AO_ANY ? cv.adagrad != 0 : OPT == AO_ADAGRAD; }
template <int OPT> __device__ __forceinline__ bool by_rowwise(const CacheView &) { return OPT == AO_ROWWISE; }

// The optimizer step on one cached row for chunk c of the row, and nothing else.
// Row-wise Adagrad's denominator for the row in `slot`: the row group adds up the squares of the
// gradient's pieces (every lane of the group calls, lanes beyond the row with zeros; the row has one
// piece per lane), the accumulator takes their mean, and the group's first lane stores it.
template <int VEC>
__device__ __forceinline__ float rowwise_rcp(const CacheView &cv, uint32_t slot, const float (&G)[VEC], float eps, uint32_t from_key, bool gone, uint32_t push_key)
{
    double ss = 0.0;
#pragma unroll
    for (int k = 0; k < VEC; ++k) ss += (double)G[k] * (double)G[k];
    for (int o = cv.geom.lanes / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o, WAVE);     // (the same tree in every lane: the same sum)
    const float a = (from_key != KEY_NONE ? cv.A[from_key] : cv.acc[slot]) + (float)(ss / (double)cv.geom.dim);
    if (threadIdx.x % cv.geom.lanes == 0) {
        if (!gone) cv.acc[slot] = a;
        if (push_key != KEY_NONE) cv.A[push_key] = a;
    }
    return fast_rcp(fast_sqrt(a) + eps);
}

// `from_key` other than KEY_NONE: the row has not been fetched yet (see apply_kernel, "fresh"): it is
// read from the global table at that key.  The result goes to the slot, unless the trim beside the update drops the row
// (gone), and to the global table at push_key, unless that is KEY_NONE (see push_key_of).
template <int VEC, int OPT>
__device__ __forceinline__ void apply_step(const CacheView &cv, uint32_t slot, int c, const double *g64, float lr, float eps, bool act,
                                           uint32_t from_key, bool gone, uint32_t push_key)
{
    using V = typename VecT<VEC>::type;
    float G[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) G[k] = act ? (float)g64[k] : 0.f;           // the fp64 sum is rounded to fp32 once
    float row_rcp = 0.f;
    if (by_rowwise<OPT>(cv)) row_rcp = rowwise_rcp<VEC>(cv, slot, G, eps, from_key, gone, push_key);
    if (!act) return;
    const bool fresh = from_key != KEY_NONE;
    V *xp = reinterpret_cast<V *>(cv.rows + (size_t)slot * cv.geom.dim) + c;
    V xv = fresh ? reinterpret_cast<const V *>(cv.W + (size_t)from_key * cv.geom.dim)[c] : *xp;
    float *x = reinterpret_cast<float *>(&xv);
    if (by_rowwise<OPT>(cv)) {
#pragma unroll
        for (int k = 0; k < VEC; ++k) x[k] = minus(x[k], lr * G[k] * row_rcp);
    } else if (by_adagrad<OPT>(cv)) {
        V *ap = reinterpret_cast<V *>(cv.acc + (size_t)slot * cv.geom.dim) + c;
        V av = fresh ? reinterpret_cast<const V *>(cv.A + (size_t)from_key * cv.geom.dim)[c] : *ap;
        float *a = reinterpret_cast<float *>(&av);
#pragma unroll
        for (int k = 0; k < VEC; ++k) { a[k] += G[k] * G[k]; x[k] = minus(x[k], lr * G[k] * fast_rcp(fast_sqrt(a[k]) + eps)); }
        if (!gone) *ap = av;
        if (push_key != KEY_NONE) reinterpret_cast<V *>(cv.A + (size_t)push_key * cv.geom.dim)[c] = av;
    } else {
#pragma unroll
        for (int k = 0; k < VEC; ++k) x[k] = minus(x[k], lr * G[k]);
    }
    if (!gone) *xp = xv;
    if (push_key != KEY_NONE) reinterpret_cast<V *>(cv.W + (size_t)push_key * cv.geom.dim)[c] = xv;     // the push
}

// Where an update puts a row besides, or instead of, its slot: the global table, if the trim beside it drops the row (TIED: any
// row of the batch, else only rows it fetched); early push: also if it fetched the row.
template <bool EARLY, bool TIED>
__device__ __forceinline__ uint32_t push_key_of(uint32_t key, uint32_t from_key, bool gone)
{
    if constexpr (TIED) return gone || (EARLY && from_key != KEY_NONE) ? key : KEY_NONE;
    return EARLY || gone ? from_key : KEY_NONE;
}

// Drops the victims among EV_SLOTS consecutive slots, EV_ITEMS per thread: erase the key, free the slot,
// raise c_g; then one row group per victim that holds updates copies its row (and accumulator)
// to the global table: Evict's push (Section 3.1).  Where a victim goes in the evicted-id list
// and (host-backed table) in the staging buffer follows from the select's per-block counts, so
// the kernel has no counter that every workgroup would have to add to: at a few nanoseconds
// per addition to one address, thousands of workgroups made those additions the kernel's
// duration.  The workgroup that holds the last victim among the rows tied at the threshold
// writes the call's counters.
struct EvictLds {
    uint32_t scan[TRIM_WAVES * 8 + 8];
    uint32_t v_slot[EV_SLOTS], v_key[EV_SLOTS], v_cg[EV_SLOTS], v_at[EV_SLOTS];
    uint32_t n_push;
};
// MANY: several workers over the table (the push adds what this worker changed to the server's row:
// three more rows in flight per victim, which the one-worker kernel does not pay registers for).
// BESIDE: runs beside the update of the batch whose lookup left the overflow (see evict_beside_update in the host code).
// The batch's rows that are victims are tied at tau = t_now (LFU: fetched ones only); those the update itself writes to
// the global table (DState::cut_slot, tied_cut), and their clock will be the present one plus one.  No other victim's clock moves.
// With a kernel less, and rows fetched and dropped by one step written once: 106496 ids 68.9 -> 60.4 us a step, 114688
// ids of 128 floats 99.8 -> 92.7, 409600 ids in bags, 256 floats, 296 -> 251.
// Runs in nblk_ workgroups of TRIM_THREADS threads; `blk` is this one's index.
template <int VEC, bool MANY, bool BESIDE>
__device__ __forceinline__ void evict_body(const CacheView &cv, const TrimPlan &tp, uint32_t blk, uint32_t nblk_)
{
    EvictLds &el = lds_as<EvictLds>();
    uint32_t *scan = el.scan, *v_slot = el.v_slot, *v_key = el.v_key, *v_cg = el.v_cg, *v_at = el.v_at;
    if (blk + 1 == nblk_) { kept_remove_victims(cv, tp, v_slot, scan); return; }
    DState *ds = cv.ds;
    const uint32_t slot0 = blk * EV_SLOTS + threadIdx.x * EV_ITEMS;
    // everything this thread may need, requested at once
    const int32_t over = ds->over;                     // snapshot taken by the select
    const uint32_t tau = ds->sel_tau;
    const uint32_t take_eq = ds->sel_take;
    uint32_t key[EV_ITEMS];
    uint4 meta[EV_ITEMS];
    load_slots<EV_ITEMS>(cv, slot0, key, meta);
    // counts over the blocks before this one (whole supers, then the blocks of this super), and over all blocks
    // (rows counted as they were fetched, and updated since: all the tied ones, if tau is their policy key)
    const bool tied_dirty = tp.fetched_dirty && tau == tp.t_now;
    uint32_t c8[8] = {0, 0, 0, 0, 0, 0, 0, 0};         // before: lt, eq, dirty lt, dirty eq;  all: dirty lt
    {
        const uint32_t nblocks = (cv.n_slots + EV_SLOTS - 1) / EV_SLOTS, nsup = (nblocks + EV_SUPER - 1) / EV_SUPER;
        const uint32_t sup = blk / EV_SUPER;
        for (uint32_t i = threadIdx.x; i < nsup; i += TRIM_THREADS) {
            const uint4 v = tp.sup_cnt[i];
            c8[4] += v.z;
            if (i < sup) { c8[0] += v.x; c8[1] += v.y; c8[2] += v.z; c8[3] += tied_dirty ? v.y : v.w; }
        }
        const uint32_t b = sup * EV_SUPER + threadIdx.x;
        if (threadIdx.x < EV_SUPER && b < blk) {
            const uint4 v = tp.blk_cnt[b];
            c8[0] += v.x; c8[1] += v.y; c8[2] += v.z; c8[3] += tied_dirty ? v.y : v.w;
        }
    }
    block_sum8(c8, scan);
    const uint32_t lt_before = c8[0], eq_before = c8[1], dlt_before = c8[2], deq_before = c8[3], dlt_total = c8[4];
    if (threadIdx.x == 0) el.n_push = 0;

    // this thread's four slots: below tau / tied with tau, in slot order
    bool lt[EV_ITEMS], eq[EV_ITEMS];
    uint32_t n_lt = 0, n_eq = 0, n_free = 0;
#pragma unroll
    for (int i = 0; i < EV_ITEMS; ++i) {
        const bool cached = key[i] != KEY_NONE && over > 0 && evictable(tp, meta[i]);
        const uint32_t pk = policy_key(meta[i]);
        lt[i] = cached && pk < tau; eq[i] = cached && pk == tau;
        n_lt += lt[i]; n_eq += eq[i];
        n_free += (slot0 + i < cv.n_slots && key[i] == KEY_NONE) ? 1u : 0u;
    }
    uint32_t tot1;
    const uint32_t ex1 = block_excl_scan<TRIM_WAVES>(n_lt | (n_eq << 16), scan, tot1);
    uint32_t eq_rank = eq_before + (ex1 >> 16);        // rank of the thread's first tied row among all tied rows
    const uint32_t eq_here = tot1 >> 16;
    bool victim[EV_ITEMS], dirty[EV_ITEMS];
    uint32_t eq_at[EV_ITEMS];
    uint32_t n_vic = 0, n_dlt = 0, n_deq_vic = 0;
#pragma unroll
    for (int i = 0; i < EV_ITEMS; ++i) {
        eq_at[i] = eq_rank;
        victim[i] = lt[i] || (eq[i] && eq_rank < take_eq);
        dirty[i] = victim[i] && (meta[i].y > meta[i].x || (BESIDE && meta[i].z == tp.t_now));
        eq_rank += eq[i];
        n_vic += victim[i]; n_dlt += dirty[i] && lt[i]; n_deq_vic += dirty[i] && eq[i];
    }
    uint32_t tot2;
    const uint32_t ex2 = block_excl_scan<TRIM_WAVES>(n_vic | (n_dlt << 16), scan, tot2);
    const uint32_t nv = tot2 & 0xFFFFu;
    // victims in earlier blocks: their rows below tau, and their tied rows up to the cut
    uint32_t ev_at = lt_before + min(eq_before, take_eq) + (ex2 & 0xFFFFu);
    uint32_t dlt_at = dlt_before + (ex2 >> 16);
    const int buf = tp.ev_slot;
#pragma unroll
    for (int i = 0; i < EV_ITEMS; ++i) {
        if (victim[i]) {
        const bool by_update = BESIDE && meta[i].z == tp.t_now;
        const uint32_t slot = slot0 + i, k = key[i], my_cc = meta[i].y + (by_update ? 1u : 0u);
        tp.ev_ids[ev_at++] = k;
        const uint32_t cg = dirty[i] ? cv.Cg[k] : 0u;
        const uint32_t early = dirty[i] && cv.early_cc ? cv.early_cc[slot] : 0u;
        if (!cv.by_position) cv.slot_of[k] = SLOT_NONE;
        cv.slot_key[slot] = KEY_NONE;
        // host-backed table: rows below tau that hold updates are staged in slot order, then one
        // place per tied victim (left empty by those without updates)
        const uint32_t stage_at = lt[i] ? dlt_at : dlt_total + eq_at[i];
        if (dirty[i]) {
            if (my_cc > cg) cv.Cg[k] = my_cc;                                 // c_g = max(c_g, c_c)
            // (pushed early by the update that fetched it, not updated since, and nobody else has pushed: the row is there already)
            const bool travelled = by_update || (early == my_cc && cg == meta[i].x);
            if (!travelled) {
                const uint32_t at = atomicAdd(&el.n_push, 1u);
                v_slot[at] = slot; v_key[at] = k; v_cg[at] = my_cc > cg ? my_cc : cg; v_at[at] = stage_at;
            }
            dlt_at += lt[i];
        } else if (cv.Cg_host && eq[i]) {
            cv.hl.keys_of(buf)[stage_at] = KEY_NONE;
        }
        }
    }
    uint32_t s2[8] = {n_free, n_deq_vic, 0, 0, 0, 0, 0, 0};
    block_sum8(s2, scan);                              // also makes the push list visible to every thread
    const uint32_t free_here = s2[0], deq_vic_here = s2[1];
    const uint32_t np = el.n_push;
    const int lanes = cv.geom.lanes;
    const int group = threadIdx.x / lanes, gl = threadIdx.x % lanes, ngroups = TRIM_THREADS / lanes;
    const RowGeom g = cv.geom;
    // Evict's push, PUSH_ROWS victims per row group at a time (all their loads before the first
    // store).  Host-backed table: the rows go to the staging buffer instead; the next Read's fetch
    // kernel (or a waiting call) sends them over the host link.
    using V = typename VecT<VEC>::type;
    if constexpr (BESIDE) {
        // (table in HBM; two victims at a time: the update's kernel has no registers for four)
        using RV = typename RawVecT<VEC>::type;
        for (uint32_t v0 = group * 2; v0 < np; v0 += ngroups * 2) {
            const uint32_t v1 = min(v0 + 1, np - 1);                 // (past the end: the last row again, the same values to the same place)
            const size_t f0 = (size_t)v_slot[v0] * g.dim, f1 = (size_t)v_slot[v1] * g.dim, t0 = (size_t)v_key[v0] * g.dim, t1 = (size_t)v_key[v1] * g.dim;
            for (int c = gl; c < g.chunks; c += g.lanes) {
                const RV x0 = reinterpret_cast<const RV *>(cv.rows + f0)[c], x1 = reinterpret_cast<const RV *>(cv.rows + f1)[c];
                if (cv.adagrad) {
                    const RV a0 = reinterpret_cast<const RV *>(cv.acc + f0)[c], a1 = reinterpret_cast<const RV *>(cv.acc + f1)[c];
                    reinterpret_cast<RV *>(cv.A + t0)[c] = a0; reinterpret_cast<RV *>(cv.A + t1)[c] = a1;
                }
                reinterpret_cast<RV *>(cv.W + t0)[c] = x0; reinterpret_cast<RV *>(cv.W + t1)[c] = x1;
            }
            if (cv.rowwise && gl == 0) { cv.A[v_key[v0]] = cv.acc[v_slot[v0]]; cv.A[v_key[v1]] = cv.acc[v_slot[v1]]; }     // (one accumulator per row)
        }
    } else {
    constexpr int PUSH_ROWS = 4;
    static_assert(PUSH_ROWS == 4, "the copy below is written out for four rows");
    const bool host = cv.Cg_host != nullptr;
    const float *src_x = cv.rows, *src_a = cv.acc;
    float *dst_x = host ? cv.hl.rows_of(buf) : cv.W, *dst_a = host ? cv.hl.acc_of(buf) : cv.A;
    for (uint32_t v0 = group * PUSH_ROWS; v0 < np; v0 += ngroups * PUSH_ROWS) {
        uint32_t from[PUSH_ROWS], to[PUSH_ROWS];
#pragma unroll
        for (int r = 0; r < PUSH_ROWS; ++r) {
            const uint32_t v = min(v0 + r, np - 1);
            from[r] = v_slot[v];
            to[r] = host ? v_at[v] : v_key[v];
            if (host && gl == 0 && v0 + r < np) {
                const uint32_t vk = v_key[v];
                cv.hl.keys_of(buf)[to[r]] = vk;
                cv.hl.cg_of(buf)[to[r]] = v_cg[v];
                cv.hl.pend[vk] = ((uint64_t)tp.push_seq << 32) | (uint64_t)to[r];
            }
        }
        const bool adagrad = cv.adagrad != 0;
        for (int c = gl; c < g.chunks; c += g.lanes) {
            V x0, x1, x2, x3, a0{}, a1{}, a2{}, a3{};
            x0 = reinterpret_cast<const V *>(src_x + (size_t)from[0] * g.dim)[c];
            x1 = reinterpret_cast<const V *>(src_x + (size_t)from[1] * g.dim)[c];
            x2 = reinterpret_cast<const V *>(src_x + (size_t)from[2] * g.dim)[c];
            x3 = reinterpret_cast<const V *>(src_x + (size_t)from[3] * g.dim)[c];
            if (adagrad) {
                a0 = reinterpret_cast<const V *>(src_a + (size_t)from[0] * g.dim)[c];
                a1 = reinterpret_cast<const V *>(src_a + (size_t)from[1] * g.dim)[c];
                a2 = reinterpret_cast<const V *>(src_a + (size_t)from[2] * g.dim)[c];
                a3 = reinterpret_cast<const V *>(src_a + (size_t)from[3] * g.dim)[c];
            }
            if (MANY) {
                // several workers: the server adds what this worker accumulated since its Fetch
                // (rows past the end repeat the last one: only the first of the repeats adds)
                const bool r1 = v0 + 1 < np, r2 = v0 + 2 < np, r3 = v0 + 3 < np;
                const V w0 = reinterpret_cast<const V *>(dst_x + (size_t)to[0] * g.dim)[c], b0 = reinterpret_cast<const V *>(cv.rows0 + (size_t)from[0] * g.dim)[c];
                const V w1 = reinterpret_cast<const V *>(dst_x + (size_t)to[1] * g.dim)[c], b1 = reinterpret_cast<const V *>(cv.rows0 + (size_t)from[1] * g.dim)[c];
                const V w2 = reinterpret_cast<const V *>(dst_x + (size_t)to[2] * g.dim)[c], b2 = reinterpret_cast<const V *>(cv.rows0 + (size_t)from[2] * g.dim)[c];
                const V w3 = reinterpret_cast<const V *>(dst_x + (size_t)to[3] * g.dim)[c], b3 = reinterpret_cast<const V *>(cv.rows0 + (size_t)from[3] * g.dim)[c];
                x0 = delta_add(w0, x0, b0);
                x1 = r1 ? delta_add(w1, x1, b1) : x0; x2 = r2 ? delta_add(w2, x2, b2) : x1; x3 = r3 ? delta_add(w3, x3, b3) : x2;
                if (adagrad) {
                    const V u0 = reinterpret_cast<const V *>(dst_a + (size_t)to[0] * g.dim)[c], d0 = reinterpret_cast<const V *>(cv.acc0 + (size_t)from[0] * g.dim)[c];
                    const V u1 = reinterpret_cast<const V *>(dst_a + (size_t)to[1] * g.dim)[c], d1 = reinterpret_cast<const V *>(cv.acc0 + (size_t)from[1] * g.dim)[c];
                    const V u2 = reinterpret_cast<const V *>(dst_a + (size_t)to[2] * g.dim)[c], d2 = reinterpret_cast<const V *>(cv.acc0 + (size_t)from[2] * g.dim)[c];
                    const V u3 = reinterpret_cast<const V *>(dst_a + (size_t)to[3] * g.dim)[c], d3 = reinterpret_cast<const V *>(cv.acc0 + (size_t)from[3] * g.dim)[c];
                    a0 = delta_add(u0, a0, d0);
                    a1 = r1 ? delta_add(u1, a1, d1) : a0; a2 = r2 ? delta_add(u2, a2, d2) : a1; a3 = r3 ? delta_add(u3, a3, d3) : a2;
                }
            }
            // rows past the end repeat the last one: the same values to the same place
            reinterpret_cast<V *>(dst_x + (size_t)to[0] * g.dim)[c] = x0;
            reinterpret_cast<V *>(dst_x + (size_t)to[1] * g.dim)[c] = x1;
            reinterpret_cast<V *>(dst_x + (size_t)to[2] * g.dim)[c] = x2;
            reinterpret_cast<V *>(dst_x + (size_t)to[3] * g.dim)[c] = x3;
            if (adagrad) {
                reinterpret_cast<V *>(dst_a + (size_t)to[0] * g.dim)[c] = a0;
                reinterpret_cast<V *>(dst_a + (size_t)to[1] * g.dim)[c] = a1;
                reinterpret_cast<V *>(dst_a + (size_t)to[2] * g.dim)[c] = a2;
                reinterpret_cast<V *>(dst_a + (size_t)to[3] * g.dim)[c] = a3;
            }
        }
        if (cv.rowwise && gl == 0) {                 // (one accumulator per row; such a table is in HBM)
#pragma unroll
            for (int r = 0; r < PUSH_ROWS; ++r) cv.A[to[r]] = cv.acc[from[r]];
        }
    }
    }
    if (threadIdx.x == 0) {
        if (free_here + nv) atomicAdd(&tp.tile_free[blk / (TRIM_TILE / EV_SLOTS)], free_here + nv);     // (zero when the trim starts; a few workgroups per tile)
        // the call's counters: written by the block that holds the last tied victim (block 0 if there is none)
        const bool closes = over <= 0 ? blk == 0
                          : (take_eq == 0 ? blk == 0 : (eq_before < take_eq && take_eq <= eq_before + eq_here));
        if (closes) {
            const uint32_t evicted = over > 0 ? (uint32_t)over : 0u;
            const uint32_t evicted_dirty = over > 0 ? dlt_total + deq_before + deq_vic_here : 0u;
            ds->ev_n[buf] = evicted;
            ds->push_n[buf] = over > 0 ? dlt_total + take_eq : 0u;
            if (evicted) {
                ds->size -= (int32_t)evicted;
                cv.last->evicted = evicted; ds->total.evicted += evicted;
                cv.last->evicted_dirty = evicted_dirty; ds->total.evicted_dirty += evicted_dirty;
            }
        }
    }
}

template <int VEC, bool RIDE, bool MANY>
__global__ __launch_bounds__(TRIM_THREADS) void trim_evict_kernel(CacheView cv, TrimPlan tp, SortStage ride, SortStage ride2)
{
    uint32_t bid = blockIdx.x, nblk = gridDim.x;
    if (RIDE && run_carried(ride, ride2, bid, nblk)) return;
    evict_body<VEC, MANY, false>(cv, tp, bid, nblk);
}

// Update + Clock (Algorithm 3) in one kernel.  A workgroup takes a tile of AP_TILE consecutive
// sorted positions, brings their keys, gradient rows' numbers and slots into LDS and lists the
// tile's segments (stretches of equal keys; a run of equal keys is one segment unless it crosses a
// tile border).  Work then goes by segment, not by position:
//   - a segment of up to AP_ROWS positions is summed by one row group, a few gradient rows (ap_batch) in
//     flight at a time, in order of position, in fp64 (the kernel is bound by reading the
//     gradients; summing wide makes a long run of a popular key lose no digits), rounded once;
//   - one of up to AP_SOLO by the row groups of one wave: contiguous shares, added through shuffles (by one row group
//     it was up to eleven rounds of loads in a row, and the kernel waits for its slowest tiles: with the run beyond the border, 106496 ids 71.3 -> 69.2 us a step,
//     60.7 -> 59.1 without a cache, 8658 ids 40.2 -> 39.0);
//   - a longer one by all row groups of the workgroup together: contiguous shares, added in group
//     order through LDS.
// A segment that is a whole run gets the optimizer step and its clock at once: no partial sum ever
// leaves the workgroup.  A run of up to AP_SOLO positions that crosses a tile border belongs to the tile it begins
// in, which sums it beyond the border; the tile it ends in passes over it (both see AP_SOLO positions on either side
// of their own and so agree on its length).  Only a longer run that crosses a border (at most two per tile) leaves one
// fp64 partial sum per tile it touches in `ApplyBorders::part`, and the tile that arrives last at
// the run's counter adds them up in tile order and applies the step: which tile is last varies,
// the order of the additions does not.  Nobody waits for anybody.
// fresh_rows: the lookup whose order this update reuses left the fetch of its missed keys' rows to
// this kernel (table in HBM, one worker): where a run's key was a miss, the row and accumulator are
// read from the global table instead of the slot; the step's result goes to the slot as always.
// Fetch and Update of Algorithms 2 and 3 in one read and one write of the row.
// MODE: AP_SORTED, the update sorted its own ids.  AP_REUSED, it reuses the preceding lookup's order: the ids must
// be the ones that order was built from; extra workgroups compare them and flag any difference, others may count
// the coming trim's rows.  AP_REUSED_EVICT, it also carries the eviction (a variant of its own, without the count, because
// its arguments and registers made every other update 2 % slower).  AP_REUSED_EVICT_TIED, the same where any row of the batch
// may be a victim (tied_cut), found ones too: LRU, and more ids than the capacity (3328 ids over 1000 rows 36.8 -> 34.8
// us a step; in the kernel above it would cost the others 2 %).
// MAXC: row pieces per lane (dim / VEC / lanes, rounded up).  OPT: the optimizer.
constexpr int AP_THREADS = 256;
constexpr int AP_SORTED = 0, AP_REUSED = 1, AP_REUSED_EVICT = 2, AP_REUSED_EVICT_TIED = 3;
// Gradient rows in flight per row group, and waves per SIMD the kernel is held to (rows of one piece
// per lane).  Tiles of 64 positions: seven waves (72 registers), so that all tiles of a batch of
// config 2's or 4's size are resident from the start, with three rows in flight (Adagrad with four keeps twelve values in
// scratch memory instead of four: 106496 ids 58.4 us a step, 57.8 with three; 40000 ids in bags of five 48.9 and 46.5) or four (SGD
// without the early push; with five 200000 ids of 32 floats 83.7 us, with four 83.0).  Tiles of 128 positions (rows of more
// than 128 floats): six waves and six rows (four with the early push); seven waves were slower there.
__host__ __device__ constexpr int ap_batch(int ap_tile, bool early, int opt) { return ap_tile == 64 ? (early || opt == AO_ADAGRAD ? 3 : 4) : (early ? 4 : 6); }
__host__ __device__ constexpr int ap_waves(int ap_tile) { return ap_tile == 64 ? 7 : 6; }
constexpr int AP_SOLO = 32;
constexpr int AP_ROWS = 8;
// Positions per tile (template parameter AP_TILE): 64 where a workgroup has eight row groups or
// more (rows up to 128 floats), 128 for wider rows, whose fewer row groups would otherwise stand
// idle beside the popular keys' long segments and pay for twice as many border crossings.
__host__ __device__ constexpr int ap_tile_for(int lanes) { return lanes <= 32 ? 64 : 128; }

// Everything below that names a position of the tile counts it from AP_SOLO positions before the tile's first.
template <int VEC, int AP_TILE> struct ApplyLds {
    static constexpr int WIN = AP_TILE + 2 * AP_SOLO;
    static_assert(WIN <= AP_THREADS && AP_TILE % WAVE == 0 && AP_SOLO * 2 == WAVE, "one thread per position of the window; those before the tile are half of its first wave, those behind it half of its last");
    double share[AP_THREADS * VEC];      // the row groups' shares of a long segment
    uint32_t key[WIN];                   // KEY_NONE where there is no valid position
    uint32_t grow[WIN];                  // gradient row of each position (tile and behind it)
    int32_t slot[WIN];                   // slot of the key, valid at run heads of the tile
    uint32_t seg_start[AP_TILE + 1];     // first position of every segment, then the end of the last
    uint32_t wave_heads[WIN / WAVE];     // segments that begin in each wave's positions
    uint64_t fresh[WIN / WAVE];          // per position: a run head whose key missed in the lookup and whose row is fetched here
    int32_t cut_slot;                    // (AP_REUSED_EVICT_TIED) the batch's rows in slots up to it are victims
    uint32_t front_open, back_open;      // a run of more than AP_SOLO positions comes in through the tile's front border / goes on behind its back border
};

// How many of the conditions cond(1), cond(2), ... hold before the first that does not; found by
// a whole wave, 64 at a time.  cond must be false from some index on.
template <typename F>
__device__ __forceinline__ uint32_t wave_count_leading(F cond)
{
    uint32_t base = 0;
    for (;;) {
        const uint64_t m = __ballot(cond(base + lane_id() + 1));
        if (~m) return base + (uint32_t)__builtin_ctzll(~m);
        base += WAVE;
    }
}

// Adds the gradient rows of tile positions [lo, hi) for row piece cidx to acc64, in order, in fp64.
// If `with_row`, the cached row (and accumulator) of `slot` is requested together with the first
// batch of gradients.
template <int VEC, int BATCH, int OPT>
__device__ __forceinline__ void add_positions(const CacheView &cv, const float *__restrict__ grads, const uint32_t *grow, uint32_t lo, uint32_t hi,
                                              int cidx, bool act, double (&acc64)[VEC], bool with_row, uint32_t slot,
                                              typename VecT<VEC>::type &xr, typename VecT<VEC>::type &ar, uint32_t from_key = KEY_NONE)
{
    using V = typename VecT<VEC>::type;
    const int dim = cv.geom.dim;
    for (uint32_t b0 = lo; b0 < hi; b0 += BATCH) {
        V v[BATCH];
#pragma unroll
        for (int r = 0; r < BATCH; ++r) {
            v[r] = V{};
            if (act && b0 + r < hi) v[r] = reinterpret_cast<const V *>(grads + (size_t)grow[b0 + r] * dim)[cidx];
        }
        if (with_row && b0 == lo && act) {
            const bool fresh = from_key != KEY_NONE;          // not fetched yet: the global row
            xr = reinterpret_cast<const V *>(fresh ? cv.W + (size_t)from_key * dim : cv.rows + (size_t)slot * dim)[cidx];
            if (by_adagrad<OPT>(cv)) ar = reinterpret_cast<const V *>(fresh ? cv.A + (size_t)from_key * dim : cv.acc + (size_t)slot * dim)[cidx];
        }
#pragma unroll
        for (int r = 0; r < BATCH; ++r) {
            const float *vf = reinterpret_cast<const float *>(&v[r]);
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc64[e] += (double)vf[e];          // zero where there is no position
        }
    }
}

template <int VEC, int BATCH, int OPT>
__device__ __forceinline__ void sum_positions(const CacheView &cv, const float *__restrict__ grads, const uint32_t *grow, uint32_t lo, uint32_t hi,
                                              int cidx, bool act, double (&acc64)[VEC], bool with_row, uint32_t slot,
                                              typename VecT<VEC>::type &xr, typename VecT<VEC>::type &ar, uint32_t from_key = KEY_NONE)
{
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc64[e] = 0.0;
    add_positions<VEC, BATCH, OPT>(cv, grads, grow, lo, hi, cidx, act, acc64, with_row, slot, xr, ar, from_key);
}

struct SegWork {
    uint32_t a, b;             // positions [a, b) of the window
    int32_t slot;
    uint32_t from_key;         // KEY_NONE, or the key whose row has not been fetched yet (fresh)
    bool gone;                 // the trim that runs beside the update drops that row
    bool is_front, is_back;    // the run began in an earlier tile / goes on in a later one
};

// A row piece's store.  STREAM: past the L2, which rows written once a step would only clear of the gradients.  Used by
// the variants that push early (rows of more than 64 floats in whole 16-byte pieces, table in HBM, one worker), the
// last step of a run over several tiles excepted.  On one box, each side's runs within 0.1 %: 114688 ids of 128 floats, SGD,
// 91.9 -> 90.8 us a step, 409600 ids in bags, 256 floats, 237.1 -> 236.7; steps of 12 million floats with SGD /
// Adagrad: rows of 68 floats 58.6 / 67.1 -> 58.7 / 66.8, 100 67.4 / 80.3 -> 67.4 / 80.0, 124 70.5 / 85.3 -> 70.4 / 84.5, 132
// 86.3 / 94.1 -> 86.6 / 94.1, 256 80.3 / 88.2 -> 79.8 / 87.4, 512 110.7 / 124.4 -> 110.6 / 124.9.
template <int VEC, bool STREAM>
__device__ __forceinline__ void store_piece(typename VecT<VEC>::type *p, const typename VecT<VEC>::type &v)
{
    using RV = typename RawVecT<VEC>::type;
    if constexpr (STREAM) {
        RV r;
        __builtin_memcpy(&r, &v, sizeof(r));
        __builtin_nontemporal_store(r, reinterpret_cast<RV *>(p));
    } else {
        *p = v;
    }
}

// The optimizer step from a row already in registers.
template <int VEC, bool EARLY, int OPT>
__device__ __forceinline__ void apply_loaded(const CacheView &cv, uint32_t slot, int cidx, const double *g64, float lr, float eps,
                                             typename VecT<VEC>::type xv, typename VecT<VEC>::type av, bool act, uint32_t from_key, bool gone, uint32_t push_key)
{
    using V = typename VecT<VEC>::type;
    float *x = reinterpret_cast<float *>(&xv), *a = reinterpret_cast<float *>(&av);
    float Gs[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) Gs[e] = act ? (float)g64[e] : 0.f;          // the fp64 sum is rounded once
    float row_rcp = 0.f;
    if (by_rowwise<OPT>(cv)) row_rcp = rowwise_rcp<VEC>(cv, slot, Gs, eps, from_key, gone, push_key);            // (every lane of the row group)
    if (!act) return;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const float G = Gs[e];
        if (by_rowwise<OPT>(cv)) x[e] = minus(x[e], lr * G * row_rcp);
        else if (by_adagrad<OPT>(cv)) { a[e] += G * G; x[e] = minus(x[e], lr * G * fast_rcp(fast_sqrt(a[e]) + eps)); }
        else x[e] = minus(x[e], lr * G);
    }
    if (!gone) {
        store_piece<VEC, EARLY>(reinterpret_cast<V *>(cv.rows + (size_t)slot * cv.geom.dim) + cidx, xv);
        if (by_adagrad<OPT>(cv)) store_piece<VEC, EARLY>(reinterpret_cast<V *>(cv.acc + (size_t)slot * cv.geom.dim) + cidx, av);
    }
    if (push_key != KEY_NONE) {
        store_piece<VEC, EARLY>(reinterpret_cast<V *>(cv.W + (size_t)push_key * cv.geom.dim) + cidx, xv);
        if (by_adagrad<OPT>(cv)) store_piece<VEC, EARLY>(reinterpret_cast<V *>(cv.A + (size_t)push_key * cv.geom.dim) + cidx, av);
    }
}

// LRU, and the batch may have more keys than the capacity: then the victims among them are the first tied ones in slot order,
// up to the slot returned (-1: none).  Found from the eviction's counts, by one wave.  The slots' keys are being erased
// by the eviction beside it, but not their metadata; a free slot's last use lies before t_now.
__device__ __forceinline__ int32_t tied_cut(const CacheView &cv, const TrimPlan &tp)
{
    const DState *ds = cv.ds;
    uint32_t take = ds->sel_take;
    if (ds->over <= 0 || ds->sel_tau != tp.t_now || !take) return -1;
    const uint32_t lane = lane_id(), nblocks = (cv.n_slots + EV_SLOTS - 1) / EV_SLOTS, nsup = (nblocks + EV_SUPER - 1) / EV_SUPER;
    uint32_t sup = 0;
    for (;; sup += WAVE) {
        const uint32_t c = sup + lane < nsup ? tp.sup_cnt[sup + lane].y : 0u, inc = wave_incl_scan(c);
        const uint64_t there = __ballot(inc >= take);
        if (there || sup + WAVE >= nsup) {
            const int at = there ? __builtin_ctzll(there) : WAVE - 1;
            take -= (uint32_t)__builtin_amdgcn_readlane((int)(inc - c), at);
            sup += (uint32_t)at;
            break;
        }
        take -= (uint32_t)__builtin_amdgcn_readlane((int)inc, WAVE - 1);
    }
    static_assert(EV_SUPER <= WAVE && EV_SLOTS == 4 * WAVE, "a block per lane, then four slots per lane");
    const uint32_t b = sup * EV_SUPER + lane, cb = lane < (uint32_t)EV_SUPER && b < nblocks ? tp.blk_cnt[b].y : 0u, incb = wave_incl_scan(cb);
    const uint64_t thereb = __ballot(incb >= take);
    const int atb = thereb ? __builtin_ctzll(thereb) : 0;
    take -= (uint32_t)__builtin_amdgcn_readlane((int)(incb - cb), atb);
    const uint32_t slot0 = (sup * EV_SUPER + (uint32_t)atb) * EV_SLOTS + 4 * lane;
    uint32_t tied[4], mine = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) { tied[q] = slot0 + q < cv.n_slots && cv.meta[slot0 + q].last_use == tp.t_now ? 1u : 0u; }
#pragma unroll
    for (int q = 0; q < 4; ++q) mine += tied[q];
    uint32_t run = wave_incl_scan(mine) - mine, cut = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) { run += tied[q]; if (tied[q] && run == take) cut = slot0 + q + 1; }
    return (int32_t)wave_sum(cut) - 1;                   // (one lane found it)
}

// What the tiles of one run tell each other inside the kernel goes through loads, stores and
// read-modify-writes of device scope, which are coherent over the whole GPU by themselves (its
// L2 caches are per XCD and ordinary stores may stay in one of them until the kernel ends).  So no
// cache has to be written back or invalidated as a device-scope fence would do, thousands of
// times per kernel: a tile waits for its own stores to be acknowledged, and only then counts
// itself as arrived.
__device__ __forceinline__ void st_device(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double ld_device(const double *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_device(int32_t *p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ int32_t ld_device(const int32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_device(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t ld_device(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void stores_acknowledged() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup"); asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

struct ApplyBorders {
    double *part;          // [tiles][2][dim]: sum of the segment that came in through the tile's front border / that leaves through its back border
    int32_t *slot;         // [tiles]: slot of the run that leaves through the tile's back border (it starts in this tile)
    uint32_t *from_key;    // [tiles]: that run's key if its row has not been fetched yet, else KEY_NONE
    uint32_t *arrived;     // [tiles]: how many tiles of the run that starts in this tile have stored their sums (zero between kernels)
    // A run over more than AP_GROUP tiles is summed in two levels (see apply_kernel).  A group is named like
    // a sum in `part`, by its first tile and the border through which the run leaves or enters that tile (a
    // run's first group starts at the run's first tile, back border; a tile may end one long run and start
    // another).  The groups' sums lie behind the tiles' sums in `part` ([tiles][2][dim] more), their counters
    // behind the runs' counters in `arrived` ([tiles][2] more): no further kernel arguments.
};
constexpr uint32_t AP_GROUP = 16;

template <int VEC, int MAXC, int MODE, int AP_TILE, bool EARLY, int OPT>
__global__ __launch_bounds__(AP_THREADS) __attribute__((amdgpu_waves_per_eu(MAXC == 1 ? ap_waves(AP_TILE) : 1))) void apply_kernel(CacheView cv, Workspace ws, ApplyBorders bd, const int64_t *__restrict__ ids,
                                                           const float *__restrict__ grads, const int64_t *__restrict__ offsets, uint32_t n_bags,
                                                           float lr, float eps, uint32_t n_ids, uint32_t work_blocks, TrimPlan tp, uint32_t trim_blocks,
                                                           SortStage ride, SortStage ride2, KernelTrace tr, int fresh_rows)
{
    using V = typename VecT<VEC>::type;
    constexpr bool VERIFY = MODE != AP_SORTED, TIED = MODE == AP_REUSED_EVICT_TIED, EVICT = MODE == AP_REUSED_EVICT || TIED;
    constexpr int BATCH = ap_batch(AP_TILE, EARLY, OPT);
    // The tiles' workgroups live longest, so they take the first places; the carried stages, the select
    // stage and the id check follow in the places they leave (the other way round the step was 1 to 2 %
    // longer on every config).
    uint32_t bid = blockIdx.x < work_blocks ? blockIdx.x + (gridDim.x - work_blocks) : blockIdx.x - work_blocks, nblk = gridDim.x;
    tr.stamp(0);
    if (run_carried(ride, ride2, bid, nblk)) { tr.role(1); tr.end(); return; }
    const uint32_t verify_blocks = VERIFY ? (n_ids + VERIFY_TILE - 1) / VERIFY_TILE : 0u;
    if (MODE != AP_SORTED) {             // extra workgroups: the eviction, or the count of the coming trim's rows
        if (bid < trim_blocks) {
            if constexpr (EVICT) evict_body<VEC, false, true>(cv, tp, bid, trim_blocks);
            else trim_count_body(cv, tp, bid, lds_as<TrimLds>());
            tr.role(2); tr.end();
            return;
        }
        bid -= trim_blocks;
    }
    if (VERIFY && bid < verify_blocks) {
        // The ids must be the ones the sorted order was built from: every position's id against the
        // sorted key, by workgroups of their own.  A difference is flagged; the update goes on.
        const uint32_t nvv = cv.ds->n_valid;
        bool bad = false;
#pragma unroll
        for (int i = 0; i < VERIFY_TILE / AP_THREADS; ++i) {
            const uint32_t j = bid * VERIFY_TILE + i * AP_THREADS + threadIdx.x;
            if (j < nvv) bad |= ids[ws.perm[j]] != (int64_t)ws.skey[j];
        }
        if (__any(bad) && lane_id() == 0) atomicOr(&cv.ds->err, ERRBIT_STATE);
        tr.role(3); tr.end();
        return;
    }
    bid -= verify_blocks;
    tr.role(4);
    const RowGeom g = cv.geom;
    const uint32_t group = threadIdx.x / g.lanes, ngroups = AP_THREADS / g.lanes;
    const int gl = threadIdx.x % g.lanes;
    const uint32_t nv = cv.ds->n_valid;
    int32_t cut_slot = EVICT && !TIED ? cv.ds->cut_slot : -1;
    auto is_gone = [&](uint32_t from_key, int32_t slot) { return TIED ? slot >= 0 && slot <= cut_slot : EVICT && from_key != KEY_NONE && slot <= cut_slot; };
    if (VERIFY && bid == 0 && threadIdx.x == 0) {
        // this call did not sort: its per-call counters start here, with the lookup's key count
        DState *ds = cv.ds;
        Counters z{};
        *cv.next_call = z;
        cv.last->n = n_ids; cv.last->unique = ds->n_unique;
        atomicAdd(&ds->total.n, (unsigned long long)n_ids);
        atomicAdd(&ds->total.unique, (unsigned long long)ds->n_unique);
        if (nv < n_ids) atomicOr(&ds->err, ERRBIT_RANGE);      // the order holds ids outside the vocabulary
    }
    ApplyLds<VEC, AP_TILE> &l = lds_as<ApplyLds<VEC, AP_TILE>>();
    const uint32_t T = bid, j0 = T * AP_TILE;
    const uint32_t *skey = ws.skey;
    constexpr uint32_t WIN = ApplyLds<VEC, AP_TILE>::WIN, W0 = AP_SOLO, WAVES = WIN / WAVE;
    bool missed = false;
    {   // the tile and what lies beside it: one position per thread
        const uint32_t i = threadIdx.x, j = j0 + i - W0;   // (wraps before the first position)
        if (i < WIN) {
            const bool in = j < n_ids, own = in && i >= W0 && i < W0 + AP_TILE;      // (not nv: that is on its way itself)
            const uint32_t k = in ? skey[j] : KEY_NONE;
            uint32_t pm = in && i >= W0 ? ws.perm[j] : 0u;
            const int32_t hs = own ? ws.head_slot[j] : SLOT_NONE;
            // fresh_rows: the lookup left the fetch of its missed keys' rows to this kernel
            missed = fresh_rows && own && ws.cls[j] == (uint8_t)CLS_MISS;
            if (offsets && in && i >= W0) pm = bag_of_position(ws.bag_of, offsets, n_bags, pm);
            l.key[i] = j < nv ? k : KEY_NONE;
            l.grow[i] = pm;
            l.slot[i] = hs;
        }
    }
    if (j0 >= nv) return;                                  // (uniform: nothing valid in this tile)
    const uint32_t cnt = min((uint32_t)AP_TILE, nv - j0);
    __syncthreads();
    uint32_t nseg = 0;
    {   // the segments, in order
        const uint32_t i = threadIdx.x, w = i / WAVE;
        bool start = false;
        uint64_t m = 0;
        uint32_t end = 0;
        if (w < WAVES) {
            const bool head = i == 0 || l.key[i] != l.key[i - 1];
            const uint64_t heads = __ballot(head);
            start = head && i >= W0 && i < W0 + cnt;       // (tile positions begin and end at half a wave)
            if (w == 0) {
                // keys ascend: a run is longer than AP_SOLO if the position AP_SOLO behind its first has its key
                // (one that began before the window is; position 0 stands for its first)
                const uint32_t first = 31u - (uint32_t)__clz((uint32_t)heads);
                const bool open = !(heads >> W0 & 1ull) && l.key[first + AP_SOLO] == l.key[W0];
                if (i == W0) start = head || open;
                if (i == 0) l.front_open = open;
            }
            if (w == WAVES - 1) {
                const uint32_t behind = (uint32_t)(heads >> W0);       // run heads behind the tile
                const bool cross = cnt == AP_TILE && !(behind & 1u);
                const uint32_t more = behind ? (uint32_t)__ffs(behind) - 1u : (uint32_t)AP_SOLO;
                const bool open = cross && l.key[W0 + AP_TILE + more - 1 - AP_SOLO] == l.key[W0 + AP_TILE - 1];
                end = W0 + cnt + (cross && !open ? more : 0u);
                if (lane_id() == 0) l.back_open = open;
            }
            m = __ballot(start);
            const uint64_t fm = __ballot(missed && head);
            if (lane_id() == 0) { l.wave_heads[w] = (uint32_t)__popcll(m); l.fresh[w] = fm; }
        }
        __syncthreads();
        uint32_t before = 0;
#pragma unroll
        for (uint32_t ww = 0; ww < WAVES; ++ww) { const uint32_t c = l.wave_heads[ww]; before += ww < w ? c : 0u; nseg += c; }
        if (start) l.seg_start[before + mask_rank(m)] = i;
        if (i == WIN - WAVE) l.seg_start[nseg] = end;
        __syncthreads();
    }
    const bool front_open = l.front_open != 0;             // the first segment's run began in an earlier tile
    const bool back_open = l.back_open != 0;               // the last one's goes on
    const size_t pstride = (size_t)g.dim;
    // Which tiles the runs that cross this tile's borders touch is asked now, by the two waves that
    // will finish them (see below), so that the answer is there when the sums are.
    const uint32_t wave = threadIdx.x / WAVE;
    const bool through = front_open && back_open && nseg == 1;
    const bool do_front = wave == 0 && front_open, do_back = wave == 1 && back_open && !through;
    uint32_t T0 = T, T1 = T;
    const uint32_t border_key = do_front ? l.key[W0] : l.key[W0 + AP_TILE - 1];
    if (TIED && wave == AP_THREADS / WAVE - 1) {
        const int32_t c = tied_cut(cv, tp);
        if (lane_id() == 0) l.cut_slot = c;
    }
    if (do_front || do_back) {
        const uint32_t key = border_key;
        if (do_front)            // tiles before this one that the run also entered through their front border
            T0 = T - 1 - wave_count_leading([&](uint32_t i) { return i < T && skey[(size_t)(T - i) * AP_TILE - 1] == key; });
        if (do_back || through)  // tiles behind this one that the run also leaves through their back border
            T1 = T + 1 + wave_count_leading([&](uint32_t i) { const uint64_t je = ((uint64_t)T + i + 1) * AP_TILE; return je < nv && skey[je] == key; });
    }
    tr.stamp(1);
    // (does any segment need the whole workgroup?  every thread looks at one)
    const bool any_long = __syncthreads_or(threadIdx.x < nseg && l.seg_start[threadIdx.x + 1] - l.seg_start[threadIdx.x] > AP_SOLO) != 0;
    if (TIED) cut_slot = l.cut_slot;

    auto seg_work = [&](uint32_t sg) {
        SegWork w;
        w.a = l.seg_start[sg]; w.b = l.seg_start[sg + 1];
        w.is_front = sg == 0 && front_open; w.is_back = sg + 1 == nseg && back_open;
        w.slot = w.is_front ? SLOT_NONE : l.slot[w.a];
        w.from_key = !w.is_front && ((l.fresh[w.a / WAVE] >> (w.a % WAVE)) & 1ull) ? l.key[w.a] : KEY_NONE;
        w.gone = is_gone(w.from_key, w.slot);
        return w;
    };
    // what is left to do once the segment's sum for row piece cidx is there
    auto finish_piece = [&](const SegWork &w, int cidx, bool act, const double (&acc64)[VEC], V xr, V ar) {
        const bool closed = !w.is_front && !w.is_back;
        if (closed) {
            if (w.slot != SLOT_NONE) apply_loaded<VEC, EARLY, OPT>(cv, (uint32_t)w.slot, cidx, acc64, lr, eps, xr, ar, act, w.from_key, w.gone, push_key_of<EARLY, TIED>(TIED ? l.key[w.a] : 0u, w.from_key, w.gone));
        } else if (act) {
            double *mine = bd.part + ((size_t)T * 2 + (w.is_front ? 0 : 1)) * pstride + (size_t)cidx * VEC;
#pragma unroll
            for (int e = 0; e < VEC; ++e) st_device(mine + e, acc64[e]);
        }
    };
    auto finish_segment = [&](const SegWork &w) {
        if (gl == 0) {
            if (w.is_back && !w.is_front) { st_device(&bd.slot[T], w.slot); st_device(&bd.from_key[T], w.from_key); }
            // Clock(k): once per key per Write; a run that goes on in later tiles takes it where it starts
            if (!w.is_front && w.slot != SLOT_NONE && !cv.direct && !w.gone) atomicAdd(&cv.meta[w.slot].cc, 1u);
        }
        if (w.is_front || w.is_back) stores_acknowledged();   // the partial sum, before this tile is counted as arrived
    };
    // segments of more than AP_ROWS and up to AP_SOLO positions: one wave each, where it holds several row groups
    const uint32_t alone = MAXC == 1 && g.lanes < WAVE ? AP_ROWS : AP_SOLO;
    if constexpr (MAXC == 1) {
        const uint32_t wave_group = lane_id() / g.lanes, wave_groups = WAVE / g.lanes;
        uint32_t count = 0;
        for (uint32_t s0 = 0; s0 < nseg; s0 += WAVE) {
            const uint32_t mine = s0 + lane_id(), len = mine < nseg ? l.seg_start[mine + 1] - l.seg_start[mine] : 0u;
            for (uint64_t todo = __ballot(len > alone && len <= AP_SOLO); todo; todo &= todo - 1) {
                if (count++ % (AP_THREADS / WAVE) != wave) continue;
                const SegWork w = seg_work(s0 + (uint32_t)__builtin_ctzll(todo));
                const bool step = !w.is_front && !w.is_back && w.slot != SLOT_NONE, act = gl < g.chunks;
                const uint32_t per = (w.b - w.a + wave_groups - 1) / wave_groups;
                const uint32_t lo = min(w.a + wave_group * per, w.b), hi = min(lo + per, w.b);
                double acc64[VEC];
                V xr{}, ar{};
                sum_positions<VEC, BATCH, OPT>(cv, grads, l.grow, lo, hi, gl, act, acc64, step && wave_group == 0, (uint32_t)w.slot, xr, ar, w.from_key);
                for (int o = g.lanes; o < WAVE; o <<= 1)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc64[e] += __shfl_xor(acc64[e], o, WAVE);
                if (wave_group == 0) { finish_piece(w, gl, act, acc64, xr, ar); finish_segment(w); }
            }
        }
    }
    {
        // the shorter ones: one row group each
        for (uint32_t sg = group; sg < nseg; sg += ngroups) {
            const SegWork w = seg_work(sg);
            if (w.b - w.a > alone) continue;
            const bool step = !w.is_front && !w.is_back && w.slot != SLOT_NONE;
#pragma unroll
            for (int q = 0; q < MAXC; ++q) {
                const int cidx = gl + q * g.lanes;
                const bool act = cidx < g.chunks;
                double acc64[VEC];
                V xr{}, ar{};
                sum_positions<VEC, BATCH, OPT>(cv, grads, l.grow, w.a, w.b, cidx, act, acc64, step, (uint32_t)w.slot, xr, ar, w.from_key);
                finish_piece(w, cidx, act, acc64, xr, ar);
            }
            finish_segment(w);
        }
    }
    tr.stamp(2);
    if (any_long) {
        // longer segments (a popular key): all row groups together, one segment at a time
        for (uint32_t sg = 0; sg < nseg; ++sg) {
            const uint32_t a = l.seg_start[sg], b = l.seg_start[sg + 1];
            if (b - a <= AP_SOLO) continue;
            const bool is_front = sg == 0 && front_open, is_back = sg + 1 == nseg && back_open;
            const int32_t slot = is_front ? SLOT_NONE : l.slot[a];
            const uint32_t from_key = !is_front && ((l.fresh[a / WAVE] >> (a % WAVE)) & 1ull) ? l.key[a] : KEY_NONE;
            const bool gone = is_gone(from_key, slot);
            const bool closed = !is_front && !is_back;
            const bool step = closed && slot != SLOT_NONE;
            const uint32_t per = (b - a + ngroups - 1) / ngroups;
            const uint32_t lo = min(a + group * per, b), hi = min(lo + per, b);
#pragma unroll
            for (int q = 0; q < MAXC; ++q) {
                const int cidx = gl + q * g.lanes;
                const bool act = cidx < g.chunks;
                double acc64[VEC];
                V xr{}, ar{};
                sum_positions<VEC, BATCH, OPT>(cv, grads, l.grow, lo, hi, cidx, act, acc64, step && group == 0, (uint32_t)slot, xr, ar, from_key);
                __syncthreads();                            // (the shares of the piece before have been read)
#pragma unroll
                for (int e = 0; e < VEC; ++e) l.share[threadIdx.x * VEC + e] = acc64[e];
                __syncthreads();
                if (group == 0) {
                    double tot[VEC];
#pragma unroll
                    for (int e = 0; e < VEC; ++e) tot[e] = 0.0;
                    for (uint32_t gi = 0; gi < ngroups; ++gi)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) tot[e] += l.share[(gi * g.lanes + gl) * VEC + e];
                    if (step) apply_loaded<VEC, EARLY, OPT>(cv, (uint32_t)slot, cidx, tot, lr, eps, xr, ar, act, from_key, gone, push_key_of<EARLY, TIED>(TIED ? l.key[a] : 0u, from_key, gone));
                    else if (!closed && act) {
                        double *mine = bd.part + ((size_t)T * 2 + (is_front ? 0 : 1)) * pstride + (size_t)cidx * VEC;
#pragma unroll
                        for (int e = 0; e < VEC; ++e) st_device(mine + e, tot[e]);
                    }
                }
            }
            if (threadIdx.x == 0) {
                if (is_back && !is_front) { st_device(&bd.slot[T], slot); st_device(&bd.from_key[T], from_key); }
                if (!is_front && slot != SLOT_NONE && !cv.direct && !gone) atomicAdd(&cv.meta[slot].cc, 1u);
            }
            if (!closed && group == 0) stores_acknowledged();
        }
    }
    tr.stamp(3);
    if (!front_open && !back_open) { tr.end(); return; }

    // Runs that cross this tile's borders.  Every tile such a run touches has stored one sum; each
    // counts itself as arrived at the run's first tile, and the one that arrives last adds the
    // sums in tile order and applies the step.  The first wave sees to the run that came in
    // through the front border, the second to the run that leaves through the back border (a tile
    // that lies inside one run has only the former).
    __syncthreads();
    tr.stamp(4);
    if (!do_front && !do_back) { tr.end(); return; }
    const uint32_t m = T1 - T0 + 1;
    // Sum of `count` stored sums, four in flight at a time, in order; where(i) is the i-th one's address for row piece 0.
    auto add_up = [&](uint32_t count, auto where, int cidx, bool act, double (&sum)[VEC]) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) sum[e] = 0.0;
        for (uint32_t i0 = 0; i0 < count; i0 += 4) {
            double part[4][VEC];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t i = i0 + u;
                const double *pp = where(i < count ? i : 0u) + (size_t)(act ? cidx : 0) * VEC;
#pragma unroll
                for (int e = 0; e < VEC; ++e) part[u][e] = i < count && act ? ld_device(pp + e) : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < VEC; ++e) sum[e] += part[u][e];
        }
    };
    // the i-th tile of the run: its first tile holds the run's sum at its back border, the others at their front border
    auto tile_sum = [&](uint32_t i) { return bd.part + ((size_t)(T0 + i) * 2 + (i == 0 ? 1 : 0)) * pstride; };
    auto arrive = [&](uint32_t *counter, uint32_t expected) {
        uint32_t last = 0;
        if (lane_id() == 0) {
            // (this tile's sums were acknowledged before)
            last = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == expected - 1 ? 1u : 0u;
            if (last) *counter = 0;                         // clean for the next kernel
        }
        return __shfl(last, 0, WAVE) != 0;
    };
    // A run over more than AP_GROUP tiles (a very popular key) would keep its last tile adding for as
    // long as the rest of the kernel takes: two levels instead.  The tile that arrives last in its
    // group of AP_GROUP consecutive tiles adds the group's sums in tile order and stores the result;
    // the group that arrives last adds the groups' results in group order.  Still a fixed order.
    const bool grouped = m > AP_GROUP;
    const uint32_t ngroups_run = (m + AP_GROUP - 1) / AP_GROUP;
    if (grouped) {
        const uint32_t first = (T - T0) / AP_GROUP * AP_GROUP;          // the group's first tile, counted from T0
        const uint32_t gs = min(AP_GROUP, m - first);
        const size_t gname = (size_t)(T0 + first) * 2 + (first == 0 ? 1 : 0);
        if (!arrive(&bd.arrived[work_blocks + gname], gs)) { tr.end(); return; }
        if (lane_id() < (uint32_t)g.lanes) {
#pragma unroll
            for (int q = 0; q < MAXC; ++q) {
                const int cidx = gl + q * g.lanes;
                const bool act = cidx < g.chunks;
                if (!act) continue;
                double sum[VEC];
                add_up(gs, [&](uint32_t i) { return tile_sum(first + i); }, cidx, act, sum);
                double *mine = bd.part + ((size_t)work_blocks * 2 + gname) * pstride + (size_t)cidx * VEC;
#pragma unroll
                for (int e = 0; e < VEC; ++e) st_device(mine + e, sum[e]);
            }
        }
        stores_acknowledged();
    }
    if (!arrive(&bd.arrived[T0], grouped ? ngroups_run : m) || lane_id() >= (uint32_t)g.lanes) { tr.end(); return; }
    const int32_t slot = ld_device(&bd.slot[T0]);           // (SLOT_NONE: a key that is not cached, flagged where the order was probed)
    const uint32_t from_key = ld_device(&bd.from_key[T0]);
#pragma unroll
    for (int q = 0; q < MAXC; ++q) {
        const int cidx = gl + q * g.lanes;
        const bool act = cidx < g.chunks;
        if (!act && !by_rowwise<OPT>(cv)) continue;                  // (row-wise Adagrad: every lane of the group takes part in the row's sum)
        double sum[VEC];
        if (grouped) add_up(ngroups_run, [&](uint32_t i) { return (const double *)bd.part + ((size_t)work_blocks * 2 + (size_t)(T0 + i * AP_GROUP) * 2 + (i == 0 ? 1 : 0)) * pstride; }, cidx, act, sum);
        else add_up(m, [&](uint32_t i) { return (const double *)tile_sum(i); }, cidx, act, sum);
        if (slot != SLOT_NONE) apply_step<VEC, OPT>(cv, (uint32_t)slot, cidx, sum, lr, eps, act, from_key, is_gone(from_key, slot), push_key_of<EARLY, TIED>(border_key, from_key, is_gone(from_key, slot)));
    }
    tr.end();
}

// The variants, compiled side by side (apply_variants.hip, fill_variants.hip): X(part, kernel arguments).
#define HET_APPLY_MODES(X, part, VEC, MAXC, TILE, EARLY, OPT)                                                   \
    X(part, VEC, MAXC, AP_SORTED, TILE, EARLY, OPT) X(part, VEC, MAXC, AP_REUSED, TILE, EARLY, OPT)              \
    X(part, VEC, MAXC, AP_REUSED_EVICT, TILE, EARLY, OPT) X(part, VEC, MAXC, AP_REUSED_EVICT_TIED, TILE, EARLY, OPT)
#define HET_APPLY_VARIANTS(X)                                                                                   \
    HET_APPLY_MODES(X, 0, 4, 1, 64, false, AO_SGD) HET_APPLY_MODES(X, 0, 4, 1, 64, false, AO_ADAGRAD)            \
    HET_APPLY_MODES(X, 0, 4, 1, 64, false, AO_ROWWISE) HET_APPLY_MODES(X, 1, 4, 1, 64, true, AO_SGD)             \
    HET_APPLY_MODES(X, 1, 4, 1, 64, true, AO_ADAGRAD)                                                            \
    HET_APPLY_MODES(X, 2, 4, 1, 128, false, AO_SGD) HET_APPLY_MODES(X, 2, 4, 1, 128, false, AO_ADAGRAD)          \
    HET_APPLY_MODES(X, 2, 4, 1, 128, false, AO_ROWWISE) HET_APPLY_MODES(X, 1, 4, 1, 128, true, AO_SGD)           \
    HET_APPLY_MODES(X, 1, 4, 1, 128, true, AO_ADAGRAD)                                                           \
    HET_APPLY_MODES(X, 3, 4, 2, 128, false, AO_ANY) HET_APPLY_MODES(X, 3, 4, 2, 128, true, AO_ANY)               \
    HET_APPLY_MODES(X, 4, 4, 4, 128, false, AO_ANY) HET_APPLY_MODES(X, 4, 4, 4, 128, true, AO_ANY)               \
    HET_APPLY_MODES(X, 5, 4, 16, 128, false, AO_ANY) HET_APPLY_MODES(X, 6, 4, 16, 128, true, AO_ANY)             \
    HET_APPLY_MODES(X, 7, 1, 1, 64, false, AO_SGD) HET_APPLY_MODES(X, 7, 1, 1, 64, false, AO_ADAGRAD)            \
    HET_APPLY_MODES(X, 7, 1, 1, 64, false, AO_ROWWISE)                                                           \
    HET_APPLY_MODES(X, 7, 1, 1, 128, false, AO_SGD) HET_APPLY_MODES(X, 7, 1, 1, 128, false, AO_ADAGRAD)          \
    HET_APPLY_MODES(X, 7, 1, 1, 128, false, AO_ROWWISE)                                                          \
    HET_APPLY_MODES(X, 3, 1, 2, 128, false, AO_ANY) HET_APPLY_MODES(X, 4, 1, 4, 128, false, AO_ANY)              \
    HET_APPLY_MODES(X, 6, 1, 16, 128, false, AO_ANY)
constexpr int HET_APPLY_PARTS = 8;
#define HET_APPLY_KERNEL(VEC, MAXC, MODE, TILE, EARLY, OPT)                                                     \
    template __global__ void apply_kernel<VEC, MAXC, MODE, TILE, EARLY, OPT>(                                     \
        CacheView, Workspace, ApplyBorders, const int64_t *__restrict__, const float *__restrict__, const int64_t *__restrict__, uint32_t, float, float, \
        uint32_t, uint32_t, TrimPlan, uint32_t, SortStage, SortStage, KernelTrace, int);

#define HET_FILL_RIDES(X, part, VEC, POOLED, TRACE) X(part, VEC, POOLED, false, TRACE) X(part, VEC, POOLED, true, TRACE)
#define HET_FILL_VARIANTS(X)                                                                                    \
    HET_FILL_RIDES(X, 0, 4, false, false) HET_FILL_RIDES(X, 0, 4, true, false) HET_FILL_RIDES(X, 0, 1, false, false) \
    HET_FILL_RIDES(X, 0, 1, true, false) HET_FILL_RIDES(X, 1, 4, false, true) HET_FILL_RIDES(X, 1, 4, true, true)  \
    HET_FILL_RIDES(X, 1, 1, false, true) HET_FILL_RIDES(X, 1, 1, true, true)
constexpr int HET_FILL_PARTS = 2;
#define HET_FILL_KERNEL(VEC, POOLED, RIDE, TRACE)                                                               \
    template __global__ void fill_gather_kernel<VEC, POOLED, RIDE, TRACE>(                                        \
        CacheView, Workspace, uint32_t, uint32_t, uint32_t, uint32_t, TrimPlan, uint32_t, float *__restrict__, const int64_t *__restrict__, uint32_t, \
        const uint32_t *__restrict__, SortStage, SortStage, uint32_t, int, uint32_t, Ahead, KernelTrace, int, uint32_t);

// flush: push every cached row that holds updates and mark it clean (c_s = c_c = c_g).
template <int VEC>
__global__ __launch_bounds__(256) void flush_kernel(CacheView cv)
{
    __shared__ uint32_t lds[4];
    const RowGeom g = cv.geom;
    const uint32_t gid = (blockIdx.x * 256u + threadIdx.x) / g.lanes;
    const int gl = threadIdx.x % g.lanes;
    const uint32_t ngroups = gridDim.x * 256u / g.lanes;
    uint32_t pushed = 0;
    for (uint32_t slot = gid; slot < cv.n_slots; slot += ngroups) {
        const uint32_t key = cv.slot_key[slot];
        if (key == KEY_NONE || cv.meta[slot].cc <= cv.meta[slot].cs) continue;
        if (cv.many) sync_row_many<VEC>(cv, key, slot, gl, true, false);
        else push_row<VEC>(cv, key, slot, gl);
        if (gl == 0) { const uint32_t cg = cv.Cg[key]; cv.meta[slot].cs = cg; cv.meta[slot].cc = cg; ++pushed; }
    }
    pushed = block_sum<4>(pushed, lds);
    if (blockIdx.x == 0 && threadIdx.x == 0) { Counters z{}; *cv.next_call = z; }
    if (threadIdx.x == 0) count2(&cv.last->flushed, &cv.ds->total.flushed, pushed);
}

// The server's side of a push by a worker that is not modelled otherwise (Section 3.1, Evict): the
// global row ids[i] takes deltas[i][:] and its clock advances by one.  One row group per id.
template <int VEC>
__global__ __launch_bounds__(256) void foreign_update_kernel(CacheView cv, const int64_t *__restrict__ ids, const float *__restrict__ deltas, uint32_t n)
{
    using V = typename VecT<VEC>::type;
    const RowGeom g = cv.geom;
    const uint32_t gid = (blockIdx.x * 256u + threadIdx.x) / g.lanes, ngroups = gridDim.x * 256u / g.lanes;
    const int gl = threadIdx.x % g.lanes;
    for (uint32_t i = gid; i < n; i += ngroups) {
        const int64_t id = ids[i];
        if (id < 0 || id >= (int64_t)cv.vocab) { if (gl == 0) atomicOr(&cv.ds->err, ERRBIT_RANGE); continue; }
        V *w = reinterpret_cast<V *>(cv.W + (size_t)id * g.dim);
        const V *d = reinterpret_cast<const V *>(deltas + (size_t)i * g.dim);
        for (int c = gl; c < g.chunks; c += g.lanes) w[c] = delta_add(w[c], d[c], V{});
        if (gl == 0) cv.Cg[id] += 1;
    }
}

// Initial free list (every slot free) and empty slots.
static __global__ __launch_bounds__(256) void init_cache_kernel(CacheView cv)
{
    const uint32_t i0 = blockIdx.x * 256u + threadIdx.x, stride = gridDim.x * 256u;
    for (uint32_t i = i0; i < cv.n_slots; i += stride) {
        cv.slot_key[i] = KEY_NONE; store_meta(cv.meta, i, 0, 0, 0, 0);
    }
    for (uint32_t i = i0; i < cv.max_ids; i += stride) cv.free_list[i] = i;
}

} // namespace het
