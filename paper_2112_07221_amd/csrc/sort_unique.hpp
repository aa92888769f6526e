// Dedup of a minibatch's ids: the "unique embedding key set" of Algorithm 1 of the paper.
//
// A stable least-significant-digit radix sort of (id, position) pairs over just the bits the
// vocabulary needs.  The result is
//   skey[j], perm[j]   ids ascending with the original position of each; equal ids keep their
//                      original order, so a key's occurrences come in increasing position.
// A run of equal keys in skey is one unique key; its first position is the key's "head".
// Ids outside [0, vocab) get the key `vocab`, which sorts behind every valid id.
//
// Up to SOLO_MAX ids: one workgroup sorts them in LDS, in one launch (sort_solo_kernel), or what other kernels
// left of their sort.
// More: one to four passes of up to 11 bits, two stages per pass: a histogram stage counts the
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

__host__ __device__ inline int solo_passes(int bits) { return (bits + SOLO_MAX_BITS - 1) / SOLO_MAX_BITS; }
__host__ __device__ inline uint32_t solo_lds_bytes(int items, int width)
{
    const uint32_t bins = 1u << width;
    return SOLO_THREADS * (uint32_t)items * 8u + SOLO_WAVES * bins * 2u + bins * 4u + SOLO_WAVES * 4u;
}

template <int ITEMS>
__global__ __launch_bounds__(SOLO_THREADS) void sort_solo_kernel(const int64_t *__restrict__ ids, const uint32_t *keys_in, const uint32_t *idx_in,
                                                                 uint32_t n, uint32_t vocab, int shift, int passes, int width,
                                                                 uint32_t *keys_out, uint32_t *idx_out)
{
    extern __shared__ __align__(16) uint32_t sort_dyn_lds[];
    const uint32_t bins = 1u << width, mask = bins - 1u, w = threadIdx.x / WAVE;
    uint32_t *xkey = sort_dyn_lds, *xpay = xkey + SOLO_THREADS * ITEMS;
    uint32_t *base = xpay + SOLO_THREADS * ITEMS, *scan = base + bins;
    uint16_t *hist = reinterpret_cast<uint16_t *>(scan + SOLO_WAVES);
    const uint32_t at0 = w * (WAVE * ITEMS) + lane_id();
    uint32_t key[ITEMS], pay[ITEMS], d[ITEMS], rank[ITEMS];
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
    for (int p = 0; p < passes; ++p) {
        for (uint32_t b = threadIdx.x; b < SOLO_WAVES * bins / 2; b += SOLO_THREADS) reinterpret_cast<uint32_t *>(hist)[b] = 0;
        __syncthreads();                                   // (also: the keys of the pass before have been read back)
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) d[it] = (key[it] >> (shift + p * width)) & mask;
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

} // namespace het
