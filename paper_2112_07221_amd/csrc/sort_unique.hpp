// Dedup of a minibatch's ids: the "unique embedding key set" of Algorithm 1 of the paper.
//
// A stable least-significant-digit radix sort of (id, position) pairs over just the bits the
// vocabulary needs.  The result is
//   skey[j], perm[j]   ids ascending with the original position of each; equal ids keep their
//                      original order, so a key's occurrences come in increasing position.
// A run of equal keys in skey is one unique key; its first position is the key's "head".
// Ids outside [0, vocab) get the key `vocab`, which sorts behind every valid id.
//
// Up to SOLO_ALONE ids: one workgroup sorts them in LDS, in one launch (sort_solo_kernel); up to SOLO_MAX what other
// kernels left of their sort.
// Up to SR_MAX ids that nobody announced: two launches, divided into ranges of keys and each sorted in LDS (SortRanges).
// More, and announced batches: one to four passes of up to 11 bits, two stages per pass: a histogram stage counts the
// pass's digit per tile of 1024 keys and per super-tile of a few tiles, a scatter stage moves the keys.
// Every workgroup of a scatter stage derives its output offsets itself from the super-tiles'
// histograms and those of the tiles before its own in its super-tile ("count at the producer, prefix
// at the consumer"); no workgroup ever waits for another one, and nothing is counted with global
// atomics (a popular id would make hundreds of them hit one address).
// A stage costs a kernel boundary and a chain of some ten LDS and barrier steps whatever its digit's
// width, so few wide passes beat many narrow ones once the offsets do not have to be added up over
// every tile; the figures are beside sort_bits_alone in the host code.
//
// A stage is a device function for workgroups of 256 or 1024 threads, not a kernel: the sort of the
// NEXT minibatch (Section 4.2: its indices are known in advance) touches no cache state, so
// its stages are carried, one per kernel, in extra workgroups of the kernels of the current
// Read and Write.  At minibatch size those kernels are bound by latency, not by throughput, and
// the sort disappears inside them; a stage nobody carried runs as a kernel of its own.
#pragma once
#include "common.hpp"

namespace het {

constexpr int SORT_THREADS = 256;                        // workgroups of the kernels that carry a stage
constexpr int SORT_THREADS_ALONE = 1024;                 // workgroups of a stage's own kernel: one key per thread
constexpr int SORT_TILE = 1024;                          // keys per workgroup of a scatter stage
constexpr int SORT_MIN_BITS = 3;                         // a histogram row is read 8 digits at a time
constexpr int SORT_MAX_BITS = 11;
constexpr int SORT_MAX_BINS = 1 << SORT_MAX_BITS;

struct SortPlan {
    uint32_t n;            // keys
    uint32_t vocab;
    uint32_t ntiles;       // ceil(n / SORT_TILE)
    uint32_t super;        // tiles per super-tile: a workgroup of a histogram stage counts one (1, 4 or 8)
    uint32_t nsupers;      // ceil(ntiles / super)
    int passes;            // 1..4
    int width;             // bits per digit (3..11)
    uint32_t *hist;        // the current pass's digit counts, two 16-bit counts per word: [ntiles][bins / 2], then [nsupers][bins / 2]
};

// One stage of a sort, as handed to the kernel that runs it.
struct SortStage {
    SortPlan sp;
    const int64_t *ids;                    // the caller's ids (read by stage 0 only)
    const uint32_t *keys_in, *idx_in;      // input of the pass (idx_in unused in pass 0: the payload is the position)
    uint32_t *keys_out, *idx_out;          // output of the pass; the first stage writes the converted ids to keys_out
    int stage;                             // 2p: histogram of pass p;  2p + 1: scatter of pass p
    uint32_t blocks;                       // workgroups the stage needs (nsupers or ntiles), 0: no stage
};

// LDS of a stage run by `threads` threads.  Histogram: 16-bit counts of a super-tile's tiles.  Scatter:
// 16-bit counts per wave, the tile's offsets, the scan's words and the 32-bit sums over the histogram's
// rows (in a carried stage those borrow the counts' place).
__host__ __device__ inline uint32_t sort_stage_lds_bytes(int width, uint32_t super, int stage, int threads)
{
    const uint32_t bins = 1u << width, waves = (uint32_t)threads / WAVE;
    const uint32_t sums = threads == SORT_THREADS ? 0u : 16u * (uint32_t)threads;
    return (stage & 1) ? waves * bins * 2u + bins * 4u + 64u + sums : super * bins * 2u;
}

__device__ __forceinline__ uint32_t id_to_key(int64_t id, uint32_t vocab)
{
    return (id >= 0 && id < (int64_t)vocab) ? (uint32_t)id : vocab;
}

// Histogram stage of pass p for one super-tile.  Pass 0 reads the ids and leaves them as 32-bit keys
// (keys_out) for its scatter stage.
template <int THREADS>
__device__ __forceinline__ void sort_hist_body(const SortStage &s, uint32_t super, uint32_t *lds)
{
    constexpr int BATCH = 4;                                      // keys a thread has on their way at a time
    const SortPlan &sp = s.sp;
    const int pass = s.stage >> 1;
    const uint32_t bins = 1u << sp.width, words = bins / 2, mask = bins - 1u, shift = (uint32_t)(pass * sp.width);
    const uint32_t first = super * sp.super * SORT_TILE, end = min(sp.n, first + sp.super * SORT_TILE);
    for (uint32_t w = threadIdx.x; w < sp.super * words; w += THREADS) lds[w] = 0;
    __syncthreads();
    for (uint32_t at = first + threadIdx.x; at < end; at += BATCH * THREADS) {
        uint32_t key[BATCH];
        if (pass == 0) {
            int64_t id[BATCH];
#pragma unroll
            for (int it = 0; it < BATCH; ++it) { const uint32_t i = at + it * THREADS; id[it] = i < end ? s.ids[i] : 0; }
#pragma unroll
            for (int it = 0; it < BATCH; ++it) key[it] = id_to_key(id[it], sp.vocab);
        } else {
#pragma unroll
            for (int it = 0; it < BATCH; ++it) { const uint32_t i = at + it * THREADS; key[it] = i < end ? s.keys_in[i] : 0u; }
        }
#pragma unroll
        for (int it = 0; it < BATCH; ++it) {
            const uint32_t i = at + it * THREADS;
            if (i < end) {
                const uint32_t d = (key[it] >> shift) & mask;
                atomicAdd(&lds[(i - first) / SORT_TILE * words + (d >> 1)], 1u << ((d & 1u) * 16u));     // (a tile's count fits 16 bits)
                if (pass == 0) s.keys_out[i] = key[it];
            }
        }
    }
    __syncthreads();
    for (uint32_t w = threadIdx.x; w < words; w += THREADS) {
        uint32_t sum = 0;
        for (uint32_t t = 0; t < sp.super; ++t) {
            const uint32_t c = lds[t * words + w], tile = super * sp.super + t;
            if (sp.super > 1 && tile < sp.ntiles) sp.hist[(size_t)tile * words + w] = c;
            sum += c;
        }
        sp.hist[(size_t)(sp.ntiles + super) * words + w] = sum;
    }
}

// Rank of every key among the keys of the same digit before it in the workgroup's keys: within the wave
// by ballots over the digit's bits, across the wave's earlier items by a running count; the counts per
// wave are left in my_hist[bins] (zero before; barriers are the caller's).
// First all the ballots (registers only, all items of a bit together), then the running counts (LDS
// only): interleaved, every item would wait for both in turn.  The counts pass between the wave's lanes
// under wavefront fences, not through a volatile pointer: that made every access a flat one that
// waits for memory (a scatter stage of 1024 keys 4.5 us, most of it these accesses).
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

// Scatter stage of pass p for one tile, stable, by the workgroup of a kernel that carries it (256 threads).
// Output offset of each digit for this tile: keys of smaller digits anywhere, plus keys of the same
// digit in earlier tiles: those of earlier super-tiles and those of its own super-tile's tiles before
// it.  A thread adds up eight consecutive digits (one 16-byte load per row, four loads in flight: more
// would cost the carrying kernels occupancy) over every RLN-th row; LDS merges the row lanes.
__device__ __forceinline__ void sort_scatter_carried(const SortStage &s, uint32_t tile, uint32_t *lds)
{
    constexpr int THREADS = SORT_THREADS, ITEMS = SORT_TILE / THREADS, WAVES = THREADS / WAVE;
    const SortPlan &sp = s.sp;
    const int pass = s.stage >> 1;
    const int width = sp.width;
    const uint32_t bins = 1u << width, mask = bins - 1u, shift = (uint32_t)(pass * width);
    const uint32_t w = threadIdx.x / WAVE;
    uint16_t *wave_hist = reinterpret_cast<uint16_t *>(lds);       // [WAVES][bins]
    uint32_t *tile_base = lds + WAVES * bins / 2;                  // [bins]
    uint32_t *scan_lds = tile_base + bins;                         // [WAVES]
    // A wave owns ITEMS * 64 consecutive keys and walks them 64 at a time, so (wave, item, lane) order is position order.
    const uint32_t at0 = tile * SORT_TILE + w * (WAVE * ITEMS) + lane_id();
    uint32_t key[ITEMS], pay[ITEMS];
    {
        uint32_t *tot = lds, *bef = lds + bins;                    // borrowed until the ranking starts
        for (uint32_t b = threadIdx.x; b < 2 * bins; b += THREADS) lds[b] = 0;
        __syncthreads();
        const uint4 *h4 = reinterpret_cast<const uint4 *>(sp.hist);
        const uint32_t octs = bins / 8;                                  // width >= 3
        const uint32_t rln = octs >= (uint32_t)THREADS ? 1u : THREADS / octs;
        const uint32_t super = tile / sp.super, rows = sp.nsupers + tile % sp.super;
        for (uint32_t item = threadIdx.x; item < octs * rln; item += THREADS) {
            const uint32_t bo = item % octs, rl = item / octs;
            uint32_t t8[8], f8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) { t8[e] = 0; f8[e] = 0; }
            for (uint32_t r0 = rl; r0 < rows; r0 += 4 * rln) {
                uint4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t r = r0 + u * rln;
                    const uint32_t row = r < sp.nsupers ? sp.ntiles + r : super * sp.super + (r - sp.nsupers);
                    v[u] = r < rows ? h4[(size_t)row * octs + bo] : make_uint4(0, 0, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t r = r0 + u * rln;
                    const uint32_t c[8] = {v[u].x & 0xFFFFu, v[u].x >> 16, v[u].y & 0xFFFFu, v[u].y >> 16,
                                           v[u].z & 0xFFFFu, v[u].z >> 16, v[u].w & 0xFFFFu, v[u].w >> 16};
                    const bool super_row = r < sp.nsupers, earlier = r < super || !super_row;
#pragma unroll
                    for (int e = 0; e < 8; ++e) { t8[e] += super_row ? c[e] : 0u; f8[e] += earlier ? c[e] : 0u; }
                }
            }
            const uint32_t b = bo * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (rln == 1) { tot[b + e] = t8[e]; bef[b + e] = f8[e]; }
                else { if (t8[e]) atomicAdd(&tot[b + e], t8[e]); if (f8[e]) atomicAdd(&bef[b + e], f8[e]); }
            }
        }
        // The keys (and payload) of this tile are requested here: the offsets' registers are free
        // again, and the loads are on their way while the digits are scanned.  (Held across the
        // whole offset computation they would cost the carrying kernel part of its occupancy.)
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; key[it] = i < sp.n ? s.keys_in[i] : 0u; }
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; pay[it] = pass == 0 ? i : (i < sp.n ? s.idx_in[i] : 0u); }
        __syncthreads();
        // exclusive scan over the digits; a thread owns PER consecutive digits
        constexpr int PER = SORT_MAX_BINS / THREADS;
        const uint32_t per = bins > (uint32_t)THREADS ? bins / THREADS : 1u, b0 = threadIdx.x * per;
        uint32_t tq[PER], fq[PER], mine = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const bool in = (uint32_t)q < per && b0 + q < bins;
            tq[q] = in ? tot[b0 + q] : 0u;
            fq[q] = in ? bef[b0 + q] : 0u;
            mine += tq[q];
        }
        uint32_t total;
        uint32_t run = block_excl_scan<WAVES>(mine, scan_lds, total);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if ((uint32_t)q < per && b0 + q < bins) tile_base[b0 + q] = run + fq[q];
            run += tq[q];
        }
        // (the scan's barriers lie between the last read of tot and bef and this)
        for (uint32_t b = threadIdx.x; b < WAVES * bins / 2; b += THREADS) lds[b] = 0;
    }
    __syncthreads();

    uint32_t d[ITEMS], rank[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { d[it] = (key[it] >> shift) & mask; valid[it] = at0 + it * WAVE < sp.n; }
    rank_in_wave<ITEMS>(d, valid, width, wave_hist + w * bins, rank);
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < bins; b += THREADS) waves_before<WAVES>(wave_hist + b, bins);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (valid[it]) {
            const uint32_t pos = tile_base[d[it]] + wave_hist[w * bins + d[it]] + rank[it];
            s.keys_out[pos] = key[it];
            s.idx_out[pos] = pay[it];
        }
    }
}

// The same by a kernel of its own: 1024 threads, one key each, registers to spare.  The histogram rows
// (two digits per thread and row, ALONE_ROWS rows in flight) are on their way while the keys are
// ranked, nothing is added through LDS atomics, and there are two barriers before the scan and one after.
constexpr int ALONE_ROWS = 16;
__device__ __forceinline__ void sort_scatter_alone(const SortStage &s, uint32_t tile, uint32_t *lds)
{
    constexpr int THREADS = SORT_THREADS_ALONE, WAVES = THREADS / WAVE;
    const SortPlan &sp = s.sp;
    const int pass = s.stage >> 1;
    const uint32_t bins = 1u << sp.width, words = bins / 2, mask = bins - 1u, shift = (uint32_t)(pass * sp.width);
    const uint32_t w = threadIdx.x / WAVE;
    const uint32_t i = tile * SORT_TILE + threadIdx.x;
    const bool in = i < sp.n;
    const uint32_t key = in ? s.keys_in[i] : 0u, pay = pass == 0 ? i : (in ? s.idx_in[i] : 0u);
    // rows of the histogram: row lane rl takes rows rl, rl + rln, ...
    const uint32_t rln = THREADS / words, col = threadIdx.x % words, rl = threadIdx.x / words;
    const uint32_t super = tile / sp.super, rows = sp.nsupers + tile % sp.super;
    auto row_word = [&](uint32_t r) { return (size_t)(r < sp.nsupers ? sp.ntiles + r : super * sp.super + (r - sp.nsupers)) * words + col; };
    uint32_t v[ALONE_ROWS];
#pragma unroll
    for (int u = 0; u < ALONE_ROWS; ++u) { const uint32_t r = rl + u * rln; v[u] = r < rows ? sp.hist[row_word(r)] : 0u; }

    uint4 *part = reinterpret_cast<uint4 *>(lds);                           // [rln][words]: totals and counts before of two digits
    uint32_t *tile_base = lds + 4 * THREADS, *scan_lds = tile_base + bins;  // [bins], [WAVES]
    uint16_t *wave_hist = reinterpret_cast<uint16_t *>(scan_lds + WAVES);   // [WAVES][bins]
    for (uint32_t b = threadIdx.x; b < WAVES * words; b += THREADS) reinterpret_cast<uint32_t *>(wave_hist)[b] = 0;
    __syncthreads();
    uint32_t d[1] = {(key >> shift) & mask}, rank[1];
    const bool valid[1] = {in};
    rank_in_wave<1>(d, valid, sp.width, wave_hist + w * bins, rank);
    uint4 sum = make_uint4(0, 0, 0, 0);
    for (uint32_t r0 = rl;;) {
#pragma unroll
        for (int u = 0; u < ALONE_ROWS; ++u) {
            const uint32_t r = r0 + u * rln, c0 = v[u] & 0xFFFFu, c1 = v[u] >> 16;
            const bool super_row = r < sp.nsupers, earlier = r < super || !super_row;
            sum.x += super_row ? c0 : 0u; sum.y += super_row ? c1 : 0u;
            sum.z += earlier ? c0 : 0u; sum.w += earlier ? c1 : 0u;
        }
        r0 += ALONE_ROWS * rln;
        if (r0 >= rows) break;
#pragma unroll
        for (int u = 0; u < ALONE_ROWS; ++u) { const uint32_t r = r0 + u * rln; v[u] = r < rows ? sp.hist[row_word(r)] : 0u; }
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    // a thread takes two neighbouring digits
    uint32_t t0 = 0, t1 = 0, f0 = 0, f1 = 0;
    if (threadIdx.x < words) {
        for (uint32_t q = 0; q < rln; ++q) {
            const uint4 p = part[q * words + threadIdx.x];
            t0 += p.x; t1 += p.y; f0 += p.z; f1 += p.w;
        }
        uint32_t c[WAVES], run = 0;                                         // the counts of the waves before each wave, both digits in a word
        uint32_t *h = reinterpret_cast<uint32_t *>(wave_hist) + threadIdx.x;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) c[ww] = h[ww * words];
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) { h[ww * words] = run; run += c[ww]; }
    }
    uint32_t total;
    const uint32_t base = block_excl_scan<WAVES>(t0 + t1, scan_lds, total);
    if (threadIdx.x < words) { tile_base[2 * threadIdx.x] = base + f0; tile_base[2 * threadIdx.x + 1] = base + t0 + f1; }
    __syncthreads();
    if (in) {
        const uint32_t pos = tile_base[d[0]] + wave_hist[w * bins + d[0]] + rank[0];
        s.keys_out[pos] = key;
        s.idx_out[pos] = pay;
    }
}

// Runs stage s for tile (super-tile) `tile`; `lds` must hold sort_stage_lds_bytes(width, stage, THREADS) bytes.
template <int THREADS>
__device__ __forceinline__ void sort_stage_body(const SortStage &s, uint32_t tile, uint32_t *lds)
{
    // (256 threads) few workgroups with a long chain of dependent steps, among the many of the carrying kernel:
    // their waves go first when a SIMD has to choose
    if (THREADS == SORT_THREADS) __builtin_amdgcn_s_setprio(3);
    if (!(s.stage & 1)) sort_hist_body<THREADS>(s, tile, lds);
    else if constexpr (THREADS == SORT_THREADS) sort_scatter_carried(s, tile, lds);
    else sort_scatter_alone(s, tile, lds);
}

// A stage nobody carried.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void sort_stage_kernel(SortStage s)
{
    extern __shared__ __align__(16) uint32_t sort_dyn_lds[];
    sort_stage_body<THREADS>(s, blockIdx.x, sort_dyn_lds);
}

// The sort of a small batch by one workgroup: the keys stay in registers, ITEMS per thread, and change
// places through LDS between the passes.  From the ids (keys_in == nullptr), or from where earlier stages
// left it: keys_in (and idx_in, or the position where that is nullptr) are in order by their lowest `shift` bits,
// and ids changed since those stages began are seen as they were then (the order check flags them).
// keys_out and idx_out may be keys_in and idx_in: every key is in a register before the first is stored.
constexpr int SOLO_THREADS = 1024;
constexpr int SOLO_WAVES = SOLO_THREADS / WAVE;
constexpr int SOLO_MAX_BITS = 9;
constexpr int SOLO_MAX_ITEMS = 8;
constexpr uint32_t SOLO_MAX = SOLO_THREADS * SOLO_MAX_ITEMS;
constexpr uint32_t SOLO_ALONE = 4 * SOLO_THREADS;        // a batch none of whose stages has run

__host__ __device__ inline int solo_passes(int bits) { return (bits + SOLO_MAX_BITS - 1) / SOLO_MAX_BITS; }
__host__ __device__ inline uint32_t solo_lds_bytes(int items, int width)
{
    const uint32_t bins = 1u << width;
    return SOLO_THREADS * (uint32_t)items * 8u + SOLO_WAVES * bins * 2u + bins * 4u + SOLO_WAVES * 4u;
}

// The passes: keys (and their payload) of list places at0 + 64 * it, in place order; `n` of them.  The digits are taken
// of key - first.  `lds` holds solo_lds_bytes(ITEMS, width) bytes.
template <int ITEMS>
__device__ __forceinline__ void solo_sort(uint32_t (&key)[ITEMS], uint32_t (&pay)[ITEMS], const bool (&valid)[ITEMS], uint32_t at0, uint32_t n,
                                          uint32_t first, int shift, int passes, int width, uint32_t *lds, uint32_t *keys_out, uint32_t *idx_out)
{
    const uint32_t bins = 1u << width, mask = bins - 1u, w = threadIdx.x / WAVE;
    uint32_t *xkey = lds, *xpay = xkey + SOLO_THREADS * ITEMS;
    uint32_t *base = xpay + SOLO_THREADS * ITEMS, *scan = base + bins;
    uint16_t *hist = reinterpret_cast<uint16_t *>(scan + SOLO_WAVES);
    uint32_t d[ITEMS], rank[ITEMS];
    for (int p = 0; p < passes; ++p) {
        for (uint32_t b = threadIdx.x; b < SOLO_WAVES * bins / 2; b += SOLO_THREADS) reinterpret_cast<uint32_t *>(hist)[b] = 0;
        __syncthreads();                                   // (also: the keys of the pass before have been read back)
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) d[it] = ((key[it] - first) >> (shift + p * width)) & mask;
        if (at0 - lane_id() < n) rank_in_wave<ITEMS>(d, valid, width, hist + w * bins, rank);     // (a wave without keys leaves its counts at zero)
        __syncthreads();
        uint32_t run = 0;
        if (threadIdx.x < bins) run = waves_before<SOLO_WAVES>(hist + threadIdx.x, bins);     // (bins <= threads)
        uint32_t total;
        const uint32_t excl = block_excl_scan<SOLO_WAVES>(run, scan, total);
        if (threadIdx.x < bins) base[threadIdx.x] = excl;
        __syncthreads();
        const bool last = p + 1 == passes;
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            if (valid[it]) {
                const uint32_t pos = base[d[it]] + hist[w * bins + d[it]] + rank[it];
                if (last) { keys_out[pos] = key[it]; idx_out[pos] = pay[it]; }
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

template <int ITEMS>
__global__ __launch_bounds__(SOLO_THREADS) void sort_solo_kernel(const int64_t *__restrict__ ids, const uint32_t *keys_in, const uint32_t *idx_in,
                                                                 uint32_t n, uint32_t vocab, int shift, int passes, int width,
                                                                 uint32_t *keys_out, uint32_t *idx_out)
{
    extern __shared__ __align__(16) uint32_t sort_dyn_lds[];
    const uint32_t at0 = threadIdx.x / WAVE * (WAVE * ITEMS) + lane_id();
    uint32_t key[ITEMS], pay[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; valid[it] = i < n; pay[it] = i; }
    if (keys_in) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = valid[it] ? keys_in[at0 + it * WAVE] : 0u;
        if (idx_in) {
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) pay[it] = valid[it] ? idx_in[at0 + it * WAVE] : 0u;
        }
    } else {
        int64_t id[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) id[it] = valid[it] ? ids[at0 + it * WAVE] : 0;
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = id_to_key(id[it], vocab);
    }
    solo_sort<ITEMS>(key, pay, valid, at0, n, 0u, shift, passes, width, sort_dyn_lds, keys_out, idx_out);
}

// The sort of a batch of middling size in two launches.  The keys are divided into ranges that hold about equally many:
// a range begins at a quantile of the order sorted before this one or, if that turns out not to divide these keys
// evenly, of a sample, which every workgroup draws for itself (the same one).  A key that fills several ranges by itself
// gets one of its own.  Where the ranges begin decides nothing but how long this takes.
// First (sort_part_kernel) every tile of 1024 keys is put in order of the ranges, in its own place, and leaves where each
// range begins in it.  Then (sort_range_kernel) a workgroup per range collects its keys from all the tiles, whose
// beginnings in the tiles add up to the range's beginning in the order, and sorts them as a small batch is sorted.
// Against four stages of the general sort that is two kernel boundaries and one pass over memory less: 26624 ids 22 -> 12.6
// us, 106496 ids 25 -> 15.7 (18.9 with cuts from the sample: the fullest range holds four times the mean).  What bounds it:
// barriers and the ballots' vector instructions.
constexpr uint32_t SR_SAMPLE = 256;                      // keys drawn
constexpr uint32_t SR_MAX_RANGES = 256;
constexpr uint32_t SR_MAX_TILES = 256;
constexpr uint32_t SR_MAX = SR_MAX_TILES * SORT_TILE;    // ids of a batch
constexpr uint32_t SR_LIST = 8 * SOLO_THREADS;           // keys a workgroup sorts at a time

struct SortRanges {
    uint32_t n, vocab, ranges, ntiles;       // ranges: a power of two
    uint32_t *cuts;                          // [ranges]: where each begins
    uint16_t *begin;                         // [ranges][ntiles]: where each begins in each tile
    uint32_t *keys, *idx;                    // the tiles in order of the ranges
    const uint32_t *known;                   // an order sorted before, or nullptr
    uint32_t n_known;
};

struct SortPartLds {
    uint32_t sample[SR_SAMPLE], rank[SR_SAMPLE], at_rank[SR_SAMPLE], cuts[SR_MAX_RANGES];
    uint32_t drawn_in[SR_MAX_RANGES];
    uint32_t base[SR_MAX_RANGES], scan[SOLO_WAVES];
    uint16_t hist[SOLO_WAVES * SR_MAX_RANGES];
};

static __global__ __launch_bounds__(SOLO_THREADS) void sort_part_kernel(const int64_t *__restrict__ ids, const uint32_t *__restrict__ keys_in, SortRanges sr)
{
    static_assert(SR_SAMPLE * 4 == SOLO_THREADS && SOLO_THREADS == SORT_TILE, "four threads find a drawn key's rank; a key per thread");
    __shared__ SortPartLds l;
    const uint32_t t = threadIdx.x, w = t / WAVE, lane = lane_id(), tile = blockIdx.x, n = sr.n;
    const uint32_t i = tile * SORT_TILE + t;
    const bool in = i < n;
    uint32_t key, drawn = 0, known = 0;
    if (sr.known && t && t < sr.ranges) known = sr.known[(uint64_t)t * sr.n_known / sr.ranges];
    {
        // (one position out of every n / SR_SAMPLE, not always the same: ids that come by fields have a period)
        uint32_t at = 0;
        if (t < SR_SAMPLE) {
            const uint32_t lo = (uint32_t)((uint64_t)t * n / SR_SAMPLE), hi = (uint32_t)((uint64_t)(t + 1) * n / SR_SAMPLE);
            at = lo + (hi > lo ? __umulhi(t * 0x9E3779B9u, hi - lo) : 0u);
        }
        if (keys_in) {
            if (t < SR_SAMPLE) drawn = keys_in[at];
            key = keys_in[in ? i : 0u];
        } else {
            int64_t d = 0;
            if (t < SR_SAMPLE) d = ids[at];
            const int64_t id = ids[in ? i : 0u];
            drawn = id_to_key(d, sr.vocab); key = id_to_key(id, sr.vocab);
        }
    }
    if (t < SR_SAMPLE) { l.sample[t] = drawn; l.rank[t] = 0; l.at_rank[t] = 0; }
    if (t < sr.ranges) { l.cuts[t] = known; l.drawn_in[t] = 0; }
    for (uint32_t b = t; b < SOLO_WAVES * sr.ranges / 2; b += SOLO_THREADS) reinterpret_cast<uint32_t *>(l.hist)[b] = 0;
    __syncthreads();
    // the range of a key: the last that begins at or below it, or, if the key fills several, the first that begins at it
    const auto range_of = [&](uint32_t k) {
        uint32_t lo = 0;
        for (uint32_t step = sr.ranges / 2; step; step /= 2) if (l.cuts[lo + step] <= k) lo += step;
        if (lo && l.cuts[lo] == k && l.cuts[lo - 1] == k) {
            uint32_t first = 0, len = lo;
            while (len) { const uint32_t half = len / 2; if (l.cuts[first + half] < k) { first += half + 1; len -= half + 1; } else len = half; }
            lo = first;
        }
        return lo;
    };
    // Cuts from an order sorted before do for keys like those: if a range of more than one key gets far more of the drawn
    // keys than its share, the drawn keys make the cuts.
    bool far_off = !sr.known;
    if (!far_off) {
        bool many = false;
        if (t < SR_SAMPLE) {
            const uint32_t r = range_of(drawn);
            const bool one_key = r + 1 < sr.ranges && l.cuts[r] == drawn && l.cuts[r + 1] == drawn;
            many = !one_key && atomicAdd(&l.drawn_in[r], 1u) >= SR_SAMPLE / sr.ranges * 2 + 8;
        }
        far_off = __syncthreads_or(many) != 0;
    }
    if (far_off) {
        {   // how many drawn keys lie below each
            const uint32_t mine = l.sample[t % SR_SAMPLE];
            const uint4 *v = reinterpret_cast<const uint4 *>(l.sample) + t / SR_SAMPLE * (SR_SAMPLE / 16);
            uint32_t r = 0;
#pragma unroll
            for (uint32_t q = 0; q < SR_SAMPLE / 16; ++q) {
                const uint4 o = v[q];
                r += (o.x < mine) + (o.y < mine) + (o.z < mine) + (o.w < mine);
            }
            atomicAdd(&l.rank[t % SR_SAMPLE], r);
        }
        __syncthreads();
        if (t < SR_SAMPLE) l.at_rank[l.rank[t]] = drawn;     // (equal keys: the same to the same place)
        __syncthreads();
        if (w == 0) {        // the drawn key of a rank: the largest at it or before it
            static_assert(SR_SAMPLE == 4 * WAVE, "four ranks to a lane");
            const uint4 v = reinterpret_cast<const uint4 *>(l.at_rank)[lane];
            uint32_t m[4];
            m[0] = v.x; m[1] = max(m[0], v.y); m[2] = max(m[1], v.z); m[3] = max(m[2], v.w);
            uint32_t top = m[3];
            top = max(top, dpp_or_zero<0x111, 0xf>(top)); top = max(top, dpp_or_zero<0x112, 0xf>(top));
            top = max(top, dpp_or_zero<0x114, 0xf>(top)); top = max(top, dpp_or_zero<0x118, 0xf>(top));
            top = max(top, dpp_or_zero<0x142, 0xa>(top)); top = max(top, dpp_or_zero<0x143, 0xc>(top));
            const uint32_t before = lane ? (uint32_t)__shfl_up(top, 1, WAVE) : 0u;
            const uint32_t each = SR_SAMPLE / sr.ranges;     // 1, 2 or 4
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t r = lane * 4 + q;
                if (r % each == 0) {
                    const uint32_t c = r ? max(before, m[q]) : 0u;
                    l.cuts[r / each] = c;
                    if (tile == 0) sr.cuts[r / each] = c;
                }
            }
        }
        __syncthreads();
    } else if (tile == 0 && t < sr.ranges) sr.cuts[t] = known;
    const uint32_t lo = range_of(key);
    uint32_t d[1] = {lo}, rank[1];
    const bool valid[1] = {in};
    const int width = 31 - __clz(sr.ranges);
    rank_in_wave<1>(d, valid, width, l.hist + w * sr.ranges, rank);
    __syncthreads();
    uint32_t run = 0;
    if (t < sr.ranges) run = waves_before<SOLO_WAVES>(l.hist + t, sr.ranges);
    uint32_t total;
    const uint32_t excl = block_excl_scan<SOLO_WAVES>(run, l.scan, total);
    if (t < sr.ranges) { l.base[t] = excl; sr.begin[(size_t)t * sr.ntiles + tile] = (uint16_t)excl; }
    __syncthreads();
    if (in) {
        const uint32_t to = tile * SORT_TILE + l.base[lo] + l.hist[w * sr.ranges + lo] + rank[0];
        sr.keys[to] = key; sr.idx[to] = i;
    }
}

struct SortRangeLds {
    uint32_t first[SR_MAX_TILES];            // of a tile's keys in this range: the list place of the first ...
    uint32_t where[SR_MAX_TILES];            // ... and where it lies, less that place
    uint32_t scan[SOLO_WAVES], wave_in[SOLO_WAVES], wave_below[SOLO_WAVES];
    uint32_t marks[SR_MAX / 32];             // (more keys than fit the list)
    uint32_t work[2 * SR_LIST + (SOLO_WAVES << SOLO_MAX_BITS) / 2 + (1 << SOLO_MAX_BITS) + SOLO_WAVES];       // the list, then the passes' (solo_lds_bytes)
};

template <int ITEMS, typename F>
__device__ __forceinline__ void sort_listed(F source, const SortRanges &sr, uint32_t m, uint32_t first, int bits, uint32_t *lds, uint32_t *keys_out, uint32_t *idx_out)
{
    const uint32_t at0 = threadIdx.x / WAVE * (WAVE * ITEMS) + lane_id();
    uint32_t key[ITEMS], pay[ITEMS], from[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { const uint32_t i = at0 + it * WAVE; valid[it] = i < m; from[it] = source(valid[it] ? i : 0u); }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) { key[it] = sr.keys[from[it]]; pay[it] = sr.idx[from[it]]; }
    const int passes = solo_passes(bits), width = max(SORT_MIN_BITS, (bits + passes - 1) / passes);
    __syncthreads();                                     // (every place has been read)
    solo_sort<ITEMS>(key, pay, valid, at0, m, first, 0, passes, width, lds, keys_out, idx_out);
}

static __global__ __launch_bounds__(SOLO_THREADS) void sort_range_kernel(SortRanges sr, uint32_t *__restrict__ keys_out, uint32_t *__restrict__ idx_out)
{
    extern __shared__ __align__(16) uint32_t sort_dyn_lds[];
    SortRangeLds &l = *reinterpret_cast<SortRangeLds *>(sort_dyn_lds);
    const uint32_t t = threadIdx.x, w = t / WAVE, lane = lane_id(), range = blockIdx.x;
    const bool last = range + 1 == sr.ranges;
    uint32_t b0 = 0, b1 = 0;
    if (t < sr.ntiles) {
        b0 = sr.begin[(size_t)range * sr.ntiles + t];
        b1 = last ? min((uint32_t)SORT_TILE, sr.n - t * SORT_TILE) : sr.begin[(size_t)(range + 1) * sr.ntiles + t];
    }
    const uint32_t a = sr.cuts[range], before = range ? sr.cuts[range - 1] : 0u, behind = last ? sr.vocab + 1u : sr.cuts[range + 1];
    const bool came_in = range && before == a, one_key = a == behind && !came_in;
    uint32_t m, below;
    const uint32_t place = block_excl_scan<SOLO_WAVES>(b1 - b0, l.scan, m);
    if (t < sr.ntiles) { l.first[t] = place; l.where[t] = t * SORT_TILE + b0 - place; }
    below = block_sum<SOLO_WAVES>(b0, l.scan);           // (its barriers make the tiles' places visible)
    if (!m) return;
    keys_out += below; idx_out += below;
    const auto source = [&](uint32_t i) {                // where list place i's key lies
        uint32_t lo = 0, hi = sr.ntiles;
        while (hi - lo > 1) { const uint32_t mid = (lo + hi) / 2; if (l.first[mid] <= i) lo = mid; else hi = mid; }
        return l.where[lo] + i;
    };
    if (one_key) {
        for (uint32_t i = t; i < m; i += SOLO_THREADS) { keys_out[i] = a; idx_out[i] = sr.idx[source(i)]; }
        return;
    }
    uint32_t cur = came_in ? a + 1 : a;
    if (m <= SR_LIST) {
        const int bits = max(1, 32 - __clz(behind - 1 - cur));
        if (m <= SOLO_THREADS) sort_listed<1>(source, sr, m, cur, bits, l.work, keys_out, idx_out);
        else if (m <= 2 * SOLO_THREADS) sort_listed<2>(source, sr, m, cur, bits, l.work, keys_out, idx_out);
        else if (m <= 4 * SOLO_THREADS) sort_listed<4>(source, sr, m, cur, bits, l.work, keys_out, idx_out);
        else sort_listed<8>(source, sr, m, cur, bits, l.work, keys_out, idx_out);
        return;
    }
    // More than a workgroup sorts at a time (the sample was far off): part after part of the range, or key by key.
    const uint32_t groups = (m + WAVE - 1) / WAVE, per_wave = (groups + SOLO_WAVES - 1) / SOLO_WAVES;
    const uint32_t g0 = min(w * per_wave, groups), g1 = min(g0 + per_wave, groups);
    while (cur < behind) {
        uint32_t hi = behind, here;
        for (;;) {
            uint32_t in = 0;
            for (uint32_t g = g0; g < g1; ++g) {
                const uint32_t i = g * WAVE + lane;
                const uint32_t key = i < m ? sr.keys[source(i)] : 0u;
                const uint64_t mark = __ballot(i < m && key - cur < hi - cur);
                in += (uint32_t)__popcll(mark);
                if (lane < 2) l.marks[2 * g + lane] = (uint32_t)(mark >> (32 * lane));
            }
            if (lane == 0) l.wave_in[w] = in;
            __syncthreads();
            here = 0;
            for (int ww = 0; ww < SOLO_WAVES; ++ww) here += l.wave_in[ww];
            if (here <= SR_LIST || hi - cur == 1) break;
            hi = cur + (hi - cur) / 2;
            __syncthreads();
        }
        const bool single = hi - cur == 1;
        uint32_t at = 0;
        for (uint32_t ww = 0; ww < w; ++ww) at += l.wave_in[ww];
        for (uint32_t g = g0; g < g1; ++g) {
            const uint64_t mark = (uint64_t)l.marks[2 * g + 1] << 32 | l.marks[2 * g];
            if (mark >> lane & 1ull) {
                const uint32_t to = at + mask_rank(mark), from = source(g * WAVE + lane);
                if (single) { keys_out[to] = cur; idx_out[to] = sr.idx[from]; }
                else l.work[to] = from;
            }
            at += (uint32_t)__popcll(mark);
        }
        __syncthreads();
        if (!single && here) sort_listed<8>([&](uint32_t i) { return l.work[i]; }, sr, here, cur, max(1, 32 - __clz(hi - 1 - cur)), l.work, keys_out, idx_out);
        keys_out += here; idx_out += here;
        cur = hi;
        __syncthreads();
    }
}

} // namespace het
