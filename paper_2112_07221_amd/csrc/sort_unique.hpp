// Dedup of a minibatch's ids: the "unique embedding key set" of Algorithm 1 of the paper.
//
// A stable sort of (id, position) pairs.  The result is
//   skey[j], perm[j]   ids ascending with the original position of each; equal ids keep their
//                      original order, so a key's occurrences come in increasing position.
// A run of equal keys in skey is one unique key; its first position is the key's "head".
// Ids outside [0, vocab) get the key `vocab`, which sorts behind every valid id.
//
// Up to SOLO_MAX ids that nobody announced: one workgroup sorts them in LDS, in one launch (sort_solo_kernel).
// More: two stages.  The keys are divided into ranges that hold about equally many.  First (part) every tile of 1024
// keys is put in order of the ranges, in its own place, and leaves where each range begins in it.  Then (range) a
// workgroup per range collects its keys from all the tiles, whose beginnings in the tiles add up to the range's beginning in
// the order, and sorts them in LDS.  No workgroup ever waits for another one, and nothing is counted with global atomics.
// A range begins at a quantile of the order sorted before this one or, if that turns out not to divide these keys evenly, of the order before
// that or of a sample, which every workgroup draws for itself (the same one), or at either.  A key that fills several ranges by itself gets
// ranges of its own, a stretch of the tiles each.  Where the ranges begin decides nothing but how long this takes, and a range that
// holds too many keys takes time in proportion to them (sort_packed, part_popular, sort_through_memory).  A step of 106496 ids, announced one
// ahead, 48.7 us; if a rare key makes up 1, 2 or 4 % of every second batch 48.7, 50.6 and 53.1 (165 to 256 where such a range's keys were
// searched again and again), of two populations in turn 49.8 (138); of 409600 ids in bags 221 us, and 223, 224, 225 (566 to 1001) and 220 (1048).
// In the place of a radix sort over the vocabulary's bits, of four to six stages: 26624 ids 22 -> 12.6 us, 106496 ids 25 -> 15.7
// (18.9 with cuts from the sample: then the fullest range holds four times the mean).  What bounds it: a kernel boundary, barriers
// and the ballots' vector instructions.
//
// A stage is a device function for workgroups of 256 or 1024 threads, not a kernel: the sort of the
// NEXT minibatch (Section 4.2: its indices are known in advance) touches no cache state, so
// its stages are carried, one per kernel, in extra workgroups of the kernels of the current
// Read and Write: the lookup's second kernel and the update.  At minibatch size those kernels are bound by latency, not by
// throughput, and the sort disappears inside them; a stage nobody carried runs as a kernel of its own.
#pragma once
#include "common.hpp"

namespace het {

constexpr int SORT_THREADS = 256;                        // workgroups of the kernels that carry a stage
constexpr int SORT_THREADS_ALONE = 1024;                 // workgroups of a stage's own kernel
constexpr int SORT_TILE = 1024;                          // keys per workgroup of a part stage
constexpr int SORT_MIN_BITS = 3;
constexpr uint32_t SORT_SAMPLE = 256;                    // keys drawn to look whether an order's cuts will do
constexpr uint32_t SORT_CUT_SAMPLE = 1024;               // keys drawn to make cuts of
constexpr uint32_t SORT_MAX_RANGES = 1024;

// How many ranges.  Carried: of up to 512 keys on average, half of what a workgroup of 256 threads sorts at a time, as long as there
// are enough (of up to 256 keys: 60000 ids 36.2 us a step instead of 35.7, 114688 75.9 instead of 75.2); beyond 524288 ids many hold more (600000 ids announced 157 us a
// step, sorted at their lookup 198; 1048576 ids 268 and 303).  Alone a workgroup sorts eight times as
// many, and ranges cost the part stage: 200000 ids in bulk 84.4 us a step with 512, 77.8 with 256.
__host__ __device__ inline uint32_t sort_ranges(uint32_t n, bool carried)
{
    const uint32_t most = carried ? 512 : (n <= 65536 ? 512 : 1024);
    uint32_t r = 64;
    while (r < SORT_MAX_RANGES && n > (r == 64 ? 256 : most) * r) r *= 2;
    return r;
}

struct SortPlan {
    uint32_t n, vocab, ranges, ntiles;       // ranges: a power of two
    uint32_t *cuts;                          // [ranges]: where each begins
    uint16_t *begin;                         // [ntiles][ranges]: where each begins in each tile
    uint32_t *keys, *idx;                    // the tiles in order of the ranges
    const uint32_t *known, *older;           // the order sorted before this one and the one before that, or nullptr
    uint32_t n_known, n_older;
};
// Words that the cuts and the beginnings of up to n ids take.
__host__ __device__ inline size_t sort_plan_words(uint32_t n) { return sort_ranges(n, true) + ((size_t)sort_ranges(n, true) * ((n + SORT_TILE - 1) / SORT_TILE) + 1) / 2; }

// One stage of a sort, as handed to the kernel that runs it.
constexpr int SORT_PART = 0, SORT_RANGE = 1, SORT_STAGES = 2;
struct SortStage {
    SortPlan sp;
    const int64_t *ids;                    // the caller's ids (part)
    uint32_t *keys_out, *idx_out;          // the order (range)
    int stage;
    uint32_t blocks;                       // workgroups the stage needs (ntiles or ranges), 0: no stage
};

__device__ __forceinline__ uint32_t id_to_key(int64_t id, uint32_t vocab)
{
    return (id >= 0 && id < (int64_t)vocab) ? (uint32_t)id : vocab;
}

// Rank of every key among the keys of the same digit before it in the workgroup's keys: within the wave
// by ballots over the digit's bits, across the wave's earlier items by a running count; the counts per
// wave are left in my_hist[bins] (zero before; barriers are the caller's).
// First all the ballots (registers only, all items of a bit together), then the running counts (LDS
// only): interleaved, every item would wait for both in turn.  The counts pass between the wave's lanes
// under wavefront fences, not through a volatile pointer: that made every access a flat one that
// waits for memory (a stage over 1024 keys 4.5 us, most of it these accesses).
template <int ITEMS>
__device__ __forceinline__ void rank_in_wave(const uint32_t (&d)[ITEMS], const bool (&valid)[ITEMS], int width, uint16_t *my_hist, uint32_t (&rank)[ITEMS])
{
    uint32_t plo[ITEMS], phi[ITEMS];    // the lanes that are valid and have the same digit
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const uint64_t v = __builtin_amdgcn_ballot_w64(valid[it]);
        plo[it] = (uint32_t)v; phi[it] = (uint32_t)(v >> 32);
    }
    for (int b = 0; b < width; ++b) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int32_t bit = __builtin_amdgcn_sbfe((int32_t)d[it], (uint32_t)b, 1u);      // the lane's bit in all places
            const uint64_t bal = __builtin_amdgcn_ballot_w64(bit != 0);
            plo[it] &= ~((uint32_t)bal ^ (uint32_t)bit);
            phi[it] &= ~((uint32_t)(bal >> 32) ^ (uint32_t)bit);
        }
    }
    uint32_t lead[ITEMS];               // for the first lane of each group of equal digits: the group's size
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        rank[it] = mask_rank(((uint64_t)phi[it] << 32) | plo[it]);
        lead[it] = (valid[it] && rank[it] == 0) ? (uint32_t)(__popc(plo[it]) + __popc(phi[it])) : 0u;
    }
    if (ITEMS == 1) {                   // (nothing before it in the wave)
        if (lead[0]) my_hist[d[0]] = (uint16_t)lead[0];
        return;
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const uint32_t before = my_hist[d[it]];
        rank[it] += before;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lead[it]) my_hist[d[it]] = (uint16_t)(before + lead[it]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Replaces a digit's counts of the waves (count[ww * bins]) by the counts of the waves before each; returns their sum.
template <int WAVES>
__device__ __forceinline__ uint32_t waves_before(uint16_t *count, uint32_t bins)
{
    uint32_t c[WAVES], run = 0;
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) c[ww] = count[ww * bins];           // (all of them before the first store)
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) { count[ww * bins] = (uint16_t)run; run += c[ww]; }
    return run;
}

// Keys a workgroup of a range stage sorts at a time, per thread and in all.
__host__ __device__ constexpr int sort_range_items(int threads) { return threads == SORT_THREADS ? 4 : 8; }
__host__ __device__ constexpr uint32_t sort_list(int threads) { return (uint32_t)(threads * sort_range_items(threads)); }

// ---- sort in LDS ------------------------------------------------------------------------------
// By one workgroup: the keys stay in registers, ITEMS per thread, and change places through LDS between the passes of a radix sort.
__host__ __device__ constexpr int solo_max_bits(int threads) { return threads == SORT_THREADS ? 8 : 9; }        // (no more digits than threads)
__host__ __device__ inline int solo_passes(int bits, int threads) { return (bits + solo_max_bits(threads) - 1) / solo_max_bits(threads); }
__host__ __device__ constexpr uint32_t solo_lds_bytes(int items, int width, int threads)
{
    return (uint32_t)(threads * items * 8 + threads / WAVE * (2 << width) + (4 << width) + threads / WAVE * 4);
}

// The passes: keys (and their payload) of list places at0 + 64 * it, in place order; `n` of them.  The digits are taken
// of key - first.  `lds` holds solo_lds_bytes(ITEMS, width, THREADS) bytes.  The order has a gap of `gap` places before its place gap_at.
template <int ITEMS, int THREADS>
__device__ __forceinline__ void solo_sort(uint32_t (&key)[ITEMS], uint32_t (&pay)[ITEMS], const bool (&valid)[ITEMS], uint32_t at0, uint32_t n,
                                          uint32_t first, int passes, int width, uint32_t *lds, uint32_t *keys_out, uint32_t *idx_out,
                                          uint32_t gap_at = 0, uint32_t gap = 0)
{
    constexpr int WAVES = THREADS / WAVE;
    const uint32_t bins = 1u << width, mask = bins - 1u, w = threadIdx.x / WAVE;
    uint32_t *xkey = lds, *xpay = xkey + THREADS * ITEMS;
    uint32_t *base = xpay + THREADS * ITEMS, *scan = base + bins;
    uint16_t *hist = reinterpret_cast<uint16_t *>(scan + WAVES);
    uint32_t d[ITEMS], rank[ITEMS];
    for (int p = 0; p < passes; ++p) {
        for (uint32_t b = threadIdx.x; b < WAVES * bins / 2; b += THREADS) reinterpret_cast<uint32_t *>(hist)[b] = 0;
        __syncthreads();                                   // (also: the keys of the pass before have been read back)
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) d[it] = ((key[it] - first) >> (p * width)) & mask;
        if (at0 - lane_id() < n) rank_in_wave<ITEMS>(d, valid, width, hist + w * bins, rank);     // (a wave without keys leaves its counts at zero)
        __syncthreads();
        uint32_t run = 0;
        if (threadIdx.x < bins) run = waves_before<WAVES>(hist + threadIdx.x, bins);     // (bins <= threads)
        uint32_t total;
        const uint32_t excl = block_excl_scan<WAVES>(run, scan, total);
        if (threadIdx.x < bins) base[threadIdx.x] = excl;
        __syncthreads();
        const bool last = p + 1 == passes;
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            if (valid[it]) {
                const uint32_t pos = base[d[it]] + hist[w * bins + d[it]] + rank[it];
                if (last) { const uint32_t to = pos < gap_at ? pos : pos + gap; keys_out[to] = key[it]; idx_out[to] = pay[it]; }
                else { xkey[pos] = key[it]; xpay[pos] = pay[it]; }
            }
        }
        if (last) return;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (valid[it]) { key[it] = xkey[at0 + it * WAVE]; pay[it] = xpay[at0 + it * WAVE]; }
    }
}

// ---- part -------------------------------------------------------------------------------------
// LDS: cuts; offsets (first: how many drawn keys a range gets); the scan's words; 16-bit counts per wave and range (first: the sort of the drawn keys).
__host__ __device__ inline uint32_t sort_part_lds_bytes(uint32_t ranges, int threads)
{
    const uint32_t waves = (uint32_t)threads / WAVE, counts = 2u * waves * ranges;
    const uint32_t drawn = threads == SORT_THREADS ? solo_lds_bytes((int)SORT_CUT_SAMPLE / threads, solo_max_bits(threads), threads) : 12u * SORT_SAMPLE;
    return 4u * (2u * ranges + waves) + (counts > drawn ? counts : drawn);
}

// A position of the j-th of `draws` equal stretches of the batch, not always the same: ids that come by fields have a period.
__device__ __forceinline__ uint32_t drawn_position(uint32_t j, uint32_t draws, uint32_t n)
{
    const uint32_t lo = (uint32_t)((uint64_t)j * n / draws), hi = (uint32_t)((uint64_t)(j + 1) * n / draws);
    return lo + (hi > lo ? __umulhi(j * 0x9E3779B9u, hi - lo) : 0u);
}

template <int THREADS>
__device__ __forceinline__ void sort_part_body(const SortStage &s, uint32_t tile, uint32_t *lds)
{
    constexpr int ITEMS = SORT_TILE / THREADS, WAVES = THREADS / WAVE;
    const SortPlan &sp = s.sp;
    const uint32_t t = threadIdx.x, w = t / WAVE, lane = lane_id(), n = sp.n, ranges = sp.ranges;
    uint32_t *cuts = lds, *base = cuts + ranges, *scan = base + ranges;
    uint16_t *hist = reinterpret_cast<uint16_t *>(scan + WAVES);
    const auto clear_hist = [&] { for (uint32_t b = t; b < WAVES * ranges / 2; b += THREADS) reinterpret_cast<uint32_t *>(hist)[b] = 0; };
    // A wave owns ITEMS * 64 consecutive keys and walks them 64 at a time, so (wave, item, lane) order is position order.
    const uint32_t at0 = tile * SORT_TILE + w * (WAVE * ITEMS) + lane;
    uint32_t key[ITEMS], drawn = 0;
    bool valid[ITEMS];
    {
        int64_t id[ITEMS], d = 0;
        if (t < SORT_SAMPLE) d = s.ids[drawn_position(t, SORT_SAMPLE, n)];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; valid[it] = i < n; id[it] = s.ids[valid[it] ? i : 0u]; }
        for (uint32_t r = t; r < ranges; r += THREADS) { cuts[r] = sp.known && r ? sp.known[(uint64_t)r * sp.n_known / ranges] : 0u; base[r] = 0; }
        drawn = id_to_key(d, sp.vocab);
        clear_hist();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = id_to_key(id[it], sp.vocab);
    }
    __syncthreads();
    // the range of a key: the last that begins at or below it, or, if the key fills several, one of these by the tile
    const auto last_at_or_below = [&](uint32_t k) {
        uint32_t lo = 0;
        for (uint32_t step = ranges / 2; step; step /= 2) if (cuts[lo + step] <= k) lo += step;
        return lo;
    };
    const auto shared = [&](uint32_t lo, uint32_t k) {
        if (lo && cuts[lo] == k && cuts[lo - 1] == k) {
            uint32_t first = 0, len = lo;
            while (len) { const uint32_t half = len / 2; if (cuts[first + half] < k) { first += half + 1; len -= half + 1; } else len = half; }
            lo = first + tile * (lo - first) / sp.ntiles;
        }
        return lo;
    };
    // Cuts from an order sorted before do for keys like those: if a range of more than one key gets far more of the drawn
    // keys than its share, cuts are made anew.  In a kernel that carries this: if the range holds, by the draws, more than a workgroup sorts
    // twice, and they are more than chance gives a range of up to two shares (106496 ids, 256 ranges: 8 of 256; measured before the order before was looked at, a step
    // with a key at 4 % of the batch 53.3 us, and 56.2 if only 11 will do).  New cuts cost such a workgroup 5 us.
    // If they will not do, those of the order before are looked at: batches of two populations in turn, a step with cuts of
    // drawn keys 56.4 us, with these 49.8 (106496 ids; of 409600 in bags 233.1 and 219.8); a new key at 4 % pays for the look (51.8 and 53.1, 223.4 and 224.5).
    bool far_off = true;
    for (const uint32_t *order = sp.known; order;) {
        bool many = false;
        if (t < SORT_SAMPLE) {
            const uint32_t r = last_at_or_below(drawn);
            const bool one_key = r && cuts[r] == drawn && cuts[r - 1] == drawn;
            const uint32_t got = one_key ? 0u : atomicAdd(&base[r], 1u) + 1u;
            const uint32_t lists = got * n / (SORT_SAMPLE * sort_list(THREADS));
            many = THREADS == SORT_THREADS ? lists > 1 && got >= SORT_SAMPLE * 3 / ranges + 5 : got >= SORT_SAMPLE * 2 / ranges + 9;
        }
        far_off = __syncthreads_or(many) != 0;
        order = far_off && order != sp.older ? sp.older : nullptr;
        if (order) {
            for (uint32_t r = t; r < ranges; r += THREADS) { cuts[r] = r ? order[(uint64_t)r * sp.n_older / ranges] : 0u; base[r] = 0; }
            __syncthreads();
        }
    }
    if (far_off) {
        uint32_t *work = scan + WAVES;
        // In a kernel that carries this, with ranges of more than a quarter of what a workgroup sorts at a time, ranges from 256 drawn keys are too
        // uneven: more are drawn.  Half of the cuts stay where the order before had them, and divide what has not changed (409600
        // ids in bags, a key at 4 %: 224 us a step, with all cuts from the drawn keys 233).
        const bool finely = THREADS == SORT_THREADS && n > sort_list(THREADS) / 4 * ranges;
        if (finely) {
            constexpr int DRAWS = SORT_CUT_SAMPLE / THREADS;
            static_assert(SORT_MAX_RANGES <= SORT_CUT_SAMPLE, "a drawn key to a range");
            uint32_t k[DRAWS], unused[DRAWS];
            int64_t id[DRAWS];
            bool all[DRAWS];
#pragma unroll
            for (int q = 0; q < DRAWS; ++q) { id[q] = s.ids[drawn_position(q * THREADS + t, SORT_CUT_SAMPLE, n)]; all[q] = true; unused[q] = 0; }
#pragma unroll
            for (int q = 0; q < DRAWS; ++q) k[q] = id_to_key(id[q], sp.vocab);
            const int bits = max(SORT_MIN_BITS, 32 - __clz(sp.vocab)), passes = solo_passes(bits, THREADS);
            solo_sort<DRAWS, THREADS>(k, unused, all, w * (WAVE * DRAWS) + lane, SORT_CUT_SAMPLE, 0u, passes, (bits + passes - 1) / passes, work, work, work + SORT_CUT_SAMPLE);
            __syncthreads();
            if (!sp.known) {
                for (uint32_t r = t; r < ranges; r += THREADS) cuts[r] = r ? work[r * (SORT_CUT_SAMPLE / ranges)] : 0u;
            } else {                                     // half of the cuts by the order before, half by the drawn keys
                const uint32_t half = ranges / 2, per = SORT_CUT_SAMPLE / half;
                for (uint32_t r = t; r < ranges; r += THREADS) {
                    const bool of_known = r < half;
                    const uint32_t cut = of_known ? cuts[2 * r] : work[(r - half) * per];
                    uint32_t at = 0;                     // how many of the others come before it (of equal ones the known)
                    for (uint32_t len = half; len;) {
                        const uint32_t mid = at + len / 2, other = of_known ? work[mid * per] : cuts[2 * mid];
                        if (of_known ? other < cut : other <= cut) { at = mid + 1; len -= len / 2 + 1; } else len /= 2;
                    }
                    base[(of_known ? r : r - half) + at] = cut;
                }
                __syncthreads();
                for (uint32_t r = t; r < ranges; r += THREADS) cuts[r] = base[r];
            }
        } else {                                         // those drawn already
            uint32_t *sample = work, *rank_of = sample + SORT_SAMPLE, *at_rank = rank_of + SORT_SAMPLE;
            if (t < SORT_SAMPLE) { sample[t] = drawn; rank_of[t] = 0; at_rank[t] = 0; }
            __syncthreads();
            constexpr uint32_t PARTS = THREADS / SORT_SAMPLE;             // threads that find one drawn key's rank
            const uint32_t mine = sample[t % SORT_SAMPLE];
            const uint4 *v = reinterpret_cast<const uint4 *>(sample) + t / SORT_SAMPLE * (SORT_SAMPLE / PARTS / 4);
            uint32_t below = 0;
#pragma unroll 8
            for (uint32_t q = 0; q < SORT_SAMPLE / PARTS / 4; ++q) {
                const uint4 o = v[q];
                below += (o.x < mine) + (o.y < mine) + (o.z < mine) + (o.w < mine);
            }
            atomicAdd(&rank_of[t % SORT_SAMPLE], below);
            __syncthreads();
            if (t < SORT_SAMPLE) at_rank[rank_of[t]] = drawn;     // (equal keys: the same to the same place)
            __syncthreads();
            if (w == 0) {        // the drawn key of a rank: the largest at it or before it
                static_assert(SORT_SAMPLE == 4 * WAVE, "four ranks to a lane");
                uint4 v = reinterpret_cast<const uint4 *>(at_rank)[lane];
                v.y = max(v.x, v.y); v.z = max(v.y, v.z); v.w = max(v.z, v.w);
                uint32_t top = v.w;
                top = max(top, dpp_or_zero<0x111, 0xf>(top)); top = max(top, dpp_or_zero<0x112, 0xf>(top));
                top = max(top, dpp_or_zero<0x114, 0xf>(top)); top = max(top, dpp_or_zero<0x118, 0xf>(top));
                top = max(top, dpp_or_zero<0x142, 0xa>(top)); top = max(top, dpp_or_zero<0x143, 0xc>(top));
                const uint32_t before = lane ? (uint32_t)__shfl_up(top, 1, WAVE) : 0u;
                reinterpret_cast<uint4 *>(at_rank)[lane] = make_uint4(max(before, v.x), max(before, v.y), max(before, v.z), max(before, v.w));
            }
            __syncthreads();
            for (uint32_t r = t; r < ranges; r += THREADS) {     // (more ranges than drawn keys: evenly between two of them)
                const uint32_t at = (uint32_t)((uint64_t)r * SORT_SAMPLE / ranges), rest = r * SORT_SAMPLE % ranges;
                const uint32_t lo = at_rank[at], hi = at + 1 < SORT_SAMPLE ? at_rank[at + 1] : sp.vocab;
                cuts[r] = r ? lo + (uint32_t)((uint64_t)(hi - lo) * rest / ranges) : 0u;
            }
        }
        __syncthreads();
        clear_hist();
        __syncthreads();
    }
    if (tile == 0) for (uint32_t r = t; r < ranges; r += THREADS) sp.cuts[r] = cuts[r];
    uint32_t d[ITEMS], rank[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) d[it] = 0;
    for (uint32_t step = ranges / 2; step; step /= 2) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) if (cuts[d[it] + step] <= key[it]) d[it] += step;
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) d[it] = shared(d[it], key[it]);
    rank_in_wave<ITEMS>(d, valid, 31 - __clz(ranges), hist + w * ranges, rank);
    __syncthreads();
    // offsets of the ranges in the tile; a thread owns `per` consecutive ones
    const uint32_t per = ranges > (uint32_t)THREADS ? ranges / THREADS : 1u, r0 = t * per;
    uint32_t mine = 0;
    if (r0 < ranges)
        for (uint32_t q = 0; q < per; ++q) { const uint32_t c = waves_before<WAVES>(hist + r0 + q, ranges); base[r0 + q] = mine; mine += c; }
    uint32_t total;
    const uint32_t excl = block_excl_scan<WAVES>(mine, scan, total);
    if (r0 < ranges)
        for (uint32_t q = 0; q < per; ++q) {
            const uint32_t at = base[r0 + q] + excl;
            base[r0 + q] = at;
            sp.begin[(size_t)tile * ranges + r0 + q] = (uint16_t)at;
        }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (valid[it]) {
            const uint32_t to = tile * SORT_TILE + base[d[it]] + hist[w * ranges + d[it]] + rank[it];
            sp.keys[to] = key[it]; sp.idx[to] = at0 + it * WAVE;
        }
    }
}

// ---- alone ------------------------------------------------------------------------------------
constexpr uint32_t SOLO_MAX = 4 * SORT_THREADS_ALONE;

// A small batch.
template <int ITEMS>
__global__ __launch_bounds__(SORT_THREADS_ALONE) void sort_solo_kernel(const int64_t *__restrict__ ids, uint32_t n, uint32_t vocab, int passes, int width,
                                                                       uint32_t *__restrict__ keys_out, uint32_t *__restrict__ idx_out)
{
    extern __shared__ __align__(16) uint32_t sort_dyn_lds[];
    const uint32_t at0 = threadIdx.x / WAVE * (WAVE * ITEMS) + lane_id();
    uint32_t key[ITEMS], pay[ITEMS];
    int64_t id[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; valid[it] = i < n; pay[it] = i; }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) id[it] = valid[it] ? ids[pay[it]] : 0;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) key[it] = id_to_key(id[it], vocab);
    solo_sort<ITEMS, SORT_THREADS_ALONE>(key, pay, valid, at0, n, 0u, passes, width, sort_dyn_lds, keys_out, idx_out);
}

// ---- range ------------------------------------------------------------------------------------
// LDS: of a tile's keys in this range, the list place of the first, and where it lies less that place; the scan's words; the
// list, then the passes'.
__host__ __device__ inline uint32_t sort_range_lds_bytes(uint32_t ntiles, int threads)
{
    return 8u * ((ntiles + 1u) / 2u * 2u) + 64u + solo_lds_bytes(sort_range_items(threads), solo_max_bits(threads), threads);
}

// The keys of a range, in the order of the tiles: where those at some list places lie.
struct RangeList {
    const uint32_t *first_of, *where;
    uint32_t ntiles, top;                                // top: the highest power of two below ntiles (0: there is one tile)
    template <int N>
    __device__ __forceinline__ void operator()(const uint32_t (&place)[N], uint32_t (&from)[N]) const
    {
        uint32_t tile[N];
#pragma unroll
        for (int q = 0; q < N; ++q) tile[q] = 0;
        for (uint32_t step = top; step; step /= 2) {     // (all the places' searches together)
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const uint32_t at = tile[q] + step;
                if (first_of[min(at, ntiles - 1)] <= place[q] && at < ntiles) tile[q] = at;
            }
        }
#pragma unroll
        for (int q = 0; q < N; ++q) from[q] = where[tile[q]] + place[q];
    }
};

template <int ITEMS, int THREADS, typename L>
__device__ __forceinline__ void sort_listed(const L &list, const SortPlan &sp, uint32_t m, uint32_t first, int bits, uint32_t *lds, uint32_t *keys_out, uint32_t *idx_out,
                                            uint32_t gap_at, uint32_t gap)
{
    const uint32_t at0 = threadIdx.x / WAVE * (WAVE * ITEMS) + lane_id();
    uint32_t key[ITEMS], pay[ITEMS], from[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; valid[it] = i < m; key[it] = valid[it] ? i : 0u; }
    list(key, from);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { key[it] = sp.keys[from[it]]; pay[it] = sp.idx[from[it]]; }
    const int passes = solo_passes(bits, THREADS), width = max(SORT_MIN_BITS, (bits + passes - 1) / passes);
    __syncthreads();                                     // (every place has been read)
    solo_sort<ITEMS, THREADS>(key, pay, valid, at0, m, first, passes, width, lds, keys_out, idx_out, gap_at, gap);
}

// Twice as many keys, of few enough bits: a word holds a key and its list place, and only words change places.  (1024 to 2048 keys in a
// kernel that carries this: 18 us, through memory 25.  Not in the sort's own kernel, which has eight times the list and whose every
// range would pay for the registers: 8000 ids 34.4 -> 35.5 us a step.)
template <int THREADS>
__device__ __forceinline__ void sort_packed(const RangeList &list, const SortPlan &sp, uint32_t m, uint32_t first, int bits, uint32_t *lds, uint32_t *keys_out, uint32_t *idx_out)
{
    constexpr int ITEMS = 2 * sort_range_items(THREADS), WAVES = THREADS / WAVE;
    constexpr uint32_t PLACES = THREADS * ITEMS;         // (a power of two)
    const int passes = solo_passes(bits, THREADS), width = max(SORT_MIN_BITS, (bits + passes - 1) / passes);
    const uint32_t bins = 1u << width, mask = bins - 1u, t = threadIdx.x, w = t / WAVE, at0 = w * (WAVE * ITEMS) + lane_id();
    uint32_t *x = lds, *base = x + PLACES, *scan = base + bins;
    uint16_t *hist = reinterpret_cast<uint16_t *>(scan + WAVES);
    uint32_t word[ITEMS], rank[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; valid[it] = i < m; word[it] = valid[it] ? i : 0u; }
    list(word, rank);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) word[it] = sp.keys[rank[it]];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) word[it] = (word[it] - first) * PLACES + at0 + it * WAVE;
    for (int p = 0; p < passes; ++p) {
        for (uint32_t b = t; b < WAVES * bins / 2; b += THREADS) reinterpret_cast<uint32_t *>(hist)[b] = 0;
        __syncthreads();                                 // (also: the words of the pass before have been read back)
        uint32_t d[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) d[it] = (word[it] / PLACES >> (p * width)) & mask;
        rank_in_wave<ITEMS>(d, valid, width, hist + w * bins, rank);
        __syncthreads();
        const uint32_t run = t < bins ? waves_before<WAVES>(hist + t, bins) : 0u;
        uint32_t total;
        const uint32_t excl = block_excl_scan<WAVES>(run, scan, total);
        if (t < bins) base[t] = excl;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) rank[it] += base[d[it]] + hist[w * bins + d[it]];
        if (p + 1 == passes) break;
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) if (valid[it]) x[rank[it]] = word[it];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) if (valid[it]) word[it] = x[at0 + it * WAVE];
    }
    uint32_t from[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (valid[it]) keys_out[rank[it]] = min(word[it] / PLACES + first, sp.vocab);      // (a key outside the range, of ids that were changed under the part stage, has lost its upper bits)
        word[it] = valid[it] ? word[it] % PLACES : 0u;
    }
    list(word, from);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) word[it] = sp.idx[from[it]];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) if (valid[it]) idx_out[rank[it]] = word[it];
}

// The most popular of the first keys of a range, if what else is in the range can be sorted at a time: its copies are put in their
// places, where the other keys lie is listed.  (4700 keys: 30 us, through memory 60.  Four keys of a thread at a time and everything read
// twice: with eight, or with the keys kept, the kernels that carry this have 100 scalar registers or more in scratch memory, and every step takes 1 % longer.)
struct SortPopular { uint32_t copies, below; };          // (copies 0: there is none)
template <int THREADS>
__device__ __forceinline__ SortPopular part_popular(const RangeList &list, const SortPlan &sp, uint32_t m, uint32_t *scan, uint32_t *others, uint32_t *keys_out, uint32_t *idx_out)
{
    constexpr int ITEMS = 4, WAVES = THREADS / WAVE, TRIED = 8;
    const uint32_t t = threadIdx.x, w = t / WAVE, first = w * (WAVE * ITEMS) + lane_id();
    uint32_t popular = 0, copies = 0, below = 0;
    for (uint32_t at0 = first; at0 - first < m; at0 += THREADS * ITEMS) {
        uint32_t key[ITEMS], from[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = min(at0 + it * WAVE, m - 1);
        list(key, from);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = sp.keys[from[it]];
        if (at0 == first) {
            if (w == 0) {
                uint32_t most = 0;
#pragma unroll
                for (int j = 0; j < TRIED; ++j) {
                    const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key[0], j * (WAVE / TRIED));
                    const uint32_t c = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(key[0] == k));
                    if (c > most) { most = c; popular = k; }
                }
                if (t == 0) { others[0] = popular; others[1] = most; }
            }
            __syncthreads();
            popular = others[0];
            const uint32_t most = others[1];
            __syncthreads();
            if (most < WAVE / 8) return {0u, 0u};        // (one in eight)
        }
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const bool in = at0 + it * WAVE < m;
            copies += in && key[it] == popular; below += in && key[it] < popular;
        }
    }
    copies = block_sum<WAVES>(copies, scan);
    below = block_sum<WAVES>(below, scan);
    if (m - copies > sort_list(THREADS)) return {0u, 0u};
    uint32_t copy_at = below, other_at = 0;
    for (uint32_t at0 = first; at0 - first < m; at0 += THREADS * ITEMS) {
        uint32_t key[ITEMS], from[ITEMS], pos[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = min(at0 + it * WAVE, m - 1);
        list(key, from);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) { key[it] = sp.keys[from[it]]; pos[it] = sp.idx[from[it]]; }
        uint32_t mine = 0, rank[ITEMS];                  // the wave's copies, and above them its other keys; of a key's kind, how many before it
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const bool in = at0 + it * WAVE < m, same = key[it] == popular;
            const uint64_t bc = __builtin_amdgcn_ballot_w64(in && same), bo = __builtin_amdgcn_ballot_w64(in && !same);
            rank[it] = same ? (mine & 0xFFFFu) + mask_rank(bc) : (mine >> 16) + mask_rank(bo);
            mine += (uint32_t)__popcll(bc) + ((uint32_t)__popcll(bo) << 16);
        }
        __syncthreads();                                 // (the words have been read)
        if (lane_id() == 0) scan[w] = mine;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) { const uint32_t c = scan[ww]; before += (uint32_t)ww < w ? c : 0u; all += c; }
        const uint32_t to_copy = copy_at + (before & 0xFFFFu), to_other = other_at + (before >> 16);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            if (at0 + it * WAVE >= m) continue;
            if (key[it] == popular) { keys_out[to_copy + rank[it]] = popular; idx_out[to_copy + rank[it]] = pos[it]; }
            else others[to_other + rank[it]] = from[it];
        }
        copy_at += all & 0xFFFFu; other_at += all >> 16;
    }
    __syncthreads();
    return {copies, below};
}

// Any number of keys: a radix sort through memory, its time in proportion to the keys whatever they are.  The range's places in the tiles
// and those in the order are this workgroup's alone, and take the keys in turn, an odd number of times.
template <int THREADS>
__device__ __forceinline__ void sort_through_memory(const RangeList &list, const SortPlan &sp, uint32_t m, uint32_t first, int bits, uint32_t *lds, uint32_t *keys_out, uint32_t *idx_out)
{
    constexpr int ITEMS = 4, COUNT = 8, WAVES = THREADS / WAVE;
    const int passes = bits <= 8 ? 1 : (bits <= 24 ? 3 : 5), width = (bits + passes - 1) / passes;
    const uint32_t bins = 1u << width, mask = bins - 1u, t = threadIdx.x, w = t / WAVE;
    uint32_t *next = lds, *base = next + passes * bins, *scan = base + bins;         // next: by pass and digit, where its next key goes
    uint16_t *hist = reinterpret_cast<uint16_t *>(scan + WAVES);
    for (uint32_t b = t; b < passes * bins; b += THREADS) next[b] = 0;
    __syncthreads();
    for (uint32_t i0 = t; i0 < m; i0 += COUNT * THREADS) {
        uint32_t key[COUNT], from[COUNT];
#pragma unroll
        for (int k = 0; k < COUNT; ++k) key[k] = min(i0 + k * THREADS, m - 1);
        list(key, from);
#pragma unroll
        for (int k = 0; k < COUNT; ++k) key[k] = sp.keys[from[k]] - first;
#pragma unroll
        for (int k = 0; k < COUNT; ++k) {
            if (i0 + k * THREADS >= m) continue;
            for (int p = 0; p < passes; ++p) {           // (the first lane's digit by one addition: mostly a popular key's)
                const uint32_t d = (key[k] >> (p * width)) & mask, d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
                const uint64_t same = __builtin_amdgcn_ballot_w64(d == d0);
                const bool leads = d == d0 && mask_rank(same) == 0;
                if (leads || d != d0) atomicAdd(&next[p * bins + d], leads ? (uint32_t)__popcll(same) : 1u);
            }
        }
    }
    for (int p = 0; p < passes; ++p) {
        const bool back = p & 1;                         // (from the order's places to the tiles')
        const uint32_t *key_in = back ? keys_out : sp.keys, *pay_in = back ? idx_out : sp.idx;
        uint32_t *key_to = back ? sp.keys : keys_out, *pay_to = back ? sp.idx : idx_out;
        uint32_t key[ITEMS], pay[ITEMS], total;
        bool valid[ITEMS];
        const auto load = [&](uint32_t at0) {
            uint32_t from[ITEMS];
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) from[it] = key[it] = min(at0 + it * WAVE, m - 1);
            if (!back) list(key, from);
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) { key[it] = key_in[from[it]]; pay[it] = pay_in[from[it]]; }
        };
        __syncthreads();                                 // (the keys have been counted, or have all moved)
        const uint32_t mine = t < bins ? next[p * bins + t] : 0u, excl = block_excl_scan<WAVES>(mine, scan, total);
        if (t < bins) next[p * bins + t] = excl;
        uint32_t at0 = w * (WAVE * ITEMS) + lane_id();
        load(at0);
        for (uint32_t c0 = 0; c0 < m; c0 += THREADS * ITEMS, at0 += THREADS * ITEMS) {
            uint32_t d[ITEMS], rank[ITEMS], k[ITEMS], q[ITEMS];
            for (uint32_t b = t; b < WAVES * bins / 2; b += THREADS) reinterpret_cast<uint32_t *>(hist)[b] = 0;
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) { k[it] = key[it]; q[it] = pay[it]; valid[it] = at0 + it * WAVE < m; d[it] = ((k[it] - first) >> (p * width)) & mask; }
            if (c0 + THREADS * ITEMS < m) load(at0 + THREADS * ITEMS);               // (under way while these are ranked)
            __syncthreads();
            rank_in_wave<ITEMS>(d, valid, width, hist + w * bins, rank);
            __syncthreads();
            if (t < bins) { const uint32_t run = waves_before<WAVES>(hist + t, bins), at = next[p * bins + t]; base[t] = at; next[p * bins + t] = at + run; }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) rank[it] = valid[it] ? rank[it] + base[d[it]] + hist[w * bins + d[it]] : 0u;
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) d[it] = rank[it];
            if (back) list(rank, d);
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) if (valid[it]) { key_to[d[it]] = k[it]; pay_to[d[it]] = q[it]; }
            __syncthreads();
        }
    }
}

template <int THREADS>
__device__ __forceinline__ void sort_range_body(const SortStage &s, uint32_t range, uint32_t *lds)
{
    constexpr int WAVES = THREADS / WAVE;
    constexpr uint32_t LIST = sort_list(THREADS);
    const SortPlan &sp = s.sp;
    uint32_t *first_of = lds, *where = first_of + (sp.ntiles + 1) / 2 * 2, *scan = where + (sp.ntiles + 1) / 2 * 2, *work = scan + 16;
    const uint32_t t = threadIdx.x;
    const bool last = range + 1 == sp.ranges;
    const uint32_t a = sp.cuts[range], before = range ? sp.cuts[range - 1] : 0u, behind = last ? sp.vocab + 1u : sp.cuts[range + 1];
    uint32_t m = 0, begin = 0;
    for (uint32_t t0 = 0; t0 < sp.ntiles; t0 += THREADS) {
        const uint32_t tile = t0 + t;
        uint32_t b0 = 0, b1 = 0, tot;
        if (tile < sp.ntiles) {
            const uint16_t *row = sp.begin + (size_t)tile * sp.ranges + range;
            b0 = row[0];
            b1 = last ? min((uint32_t)SORT_TILE, sp.n - tile * SORT_TILE) : row[1];
        }
        const uint32_t place = m + block_excl_scan<WAVES>(b1 - b0, scan, tot);
        if (tile < sp.ntiles) { first_of[tile] = place; where[tile] = tile * SORT_TILE + b0 - place; }
        m += tot; begin += b0;
    }
    begin = block_sum<WAVES>(begin, scan);               // (its barriers make the tiles' places visible)
    if (!m) return;
    const RangeList list{first_of, where, sp.ntiles, sp.ntiles > 1 ? 1u << (31 - __clz(sp.ntiles - 1)) : 0u};
    uint32_t *keys_out = s.keys_out + begin, *idx_out = s.idx_out + begin;
    const uint32_t cur = range && before == a ? a + 1 : a;         // (key a has ranges of its own before this one)
    if (a == behind) {                                   // this is one
        constexpr int COPY = 8;
        for (uint32_t i0 = t; i0 < m; i0 += COPY * THREADS) {
            uint32_t from[COPY], pos[COPY];
#pragma unroll
            for (int k = 0; k < COPY; ++k) pos[k] = min(i0 + k * THREADS, m - 1);
            list(pos, from);
#pragma unroll
            for (int k = 0; k < COPY; ++k) pos[k] = sp.idx[from[k]];
#pragma unroll
            for (int k = 0; k < COPY; ++k) if (i0 + k * THREADS < m) { keys_out[i0 + k * THREADS] = a; idx_out[i0 + k * THREADS] = pos[k]; }
        }
        return;
    }
    const int bits = max(1, 32 - __clz(behind - 1 - cur));
    const auto sort = [&](const auto &which, uint32_t count, uint32_t gap_at, uint32_t gap) {
        if constexpr (THREADS == SORT_THREADS) {
            if (count <= 2 * THREADS) sort_listed<2, THREADS>(which, sp, count, cur, bits, work, keys_out, idx_out, gap_at, gap);
            else sort_listed<4, THREADS>(which, sp, count, cur, bits, work, keys_out, idx_out, gap_at, gap);
        } else {
            if (count <= THREADS) sort_listed<1, THREADS>(which, sp, count, cur, bits, work, keys_out, idx_out, gap_at, gap);
            else if (count <= 2 * THREADS) sort_listed<2, THREADS>(which, sp, count, cur, bits, work, keys_out, idx_out, gap_at, gap);
            else if (count <= 4 * THREADS) sort_listed<4, THREADS>(which, sp, count, cur, bits, work, keys_out, idx_out, gap_at, gap);
            else sort_listed<8, THREADS>(which, sp, count, cur, bits, work, keys_out, idx_out, gap_at, gap);
        }
    };
    if (m <= LIST) { sort(list, m, 0u, 0u); return; }
    if (THREADS == SORT_THREADS && m <= 2 * LIST && bits + 32 - __clz(2 * LIST - 1) <= 32) { sort_packed<THREADS>(list, sp, m, cur, bits, work, keys_out, idx_out); return; }
    const SortPopular pop = part_popular<THREADS>(list, sp, m, scan, work, keys_out, idx_out);
    if (!pop.copies) sort_through_memory<THREADS>(list, sp, m, cur, bits, work, keys_out, idx_out);
    else if (pop.copies < m)
        sort([&](const auto &place, auto &from) { for (uint32_t q = 0; q < sizeof(place) / 4; ++q) from[q] = work[place[q]]; }, m - pop.copies, pop.below, pop.copies);
}

// ---- stages -----------------------------------------------------------------------------------
__host__ __device__ inline uint32_t sort_stage_lds_bytes(const SortStage &s, int threads)
{
    return s.stage == SORT_PART ? sort_part_lds_bytes(s.sp.ranges, threads) : sort_range_lds_bytes(s.sp.ntiles, threads);
}

// Runs stage s for tile or range `item`; `lds` must hold sort_stage_lds_bytes(s, THREADS) bytes.
template <int THREADS>
__device__ __forceinline__ void sort_stage_body(const SortStage &s, uint32_t item, uint32_t *lds)
{
    // (256 threads) few workgroups with a long chain of dependent steps, among the many of the carrying kernel:
    // their waves go first when a SIMD has to choose
    if (THREADS == SORT_THREADS) __builtin_amdgcn_s_setprio(3);
    if (s.stage == SORT_PART) sort_part_body<THREADS>(s, item, lds);
    else sort_range_body<THREADS>(s, item, lds);
}

// Stages nobody carried.
static __global__ __launch_bounds__(SORT_THREADS_ALONE) void sort_part_kernel(SortStage s)
{
    extern __shared__ __align__(16) uint32_t sort_dyn_lds[];
    sort_part_body<SORT_THREADS_ALONE>(s, blockIdx.x, sort_dyn_lds);
}
static __global__ __launch_bounds__(SORT_THREADS_ALONE) void sort_range_kernel(SortStage s)
{
    extern __shared__ __align__(16) uint32_t sort_dyn_lds[];
    sort_range_body<SORT_THREADS_ALONE>(s, blockIdx.x, sort_dyn_lds);
}

} // namespace het
