// Shared device-side definitions of the embedding-cache kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace het {

constexpr int WAVE = 64;
constexpr uint32_t KEY_NONE = 0xFFFFFFFFu;   // free slot / no key
constexpr int32_t SLOT_NONE = -1;

constexpr uint32_t ERRBIT_RANGE = 1u;        // an id outside [0, vocab)
constexpr uint32_t ERRBIT_STATE = 2u;        // update of a key that is not cached

constexpr int CLS_HIT = 0, CLS_STALE = 1, CLS_MISS = 2;

// Counters of one call, mirrored by het_counters in the public header.
struct Counters {
    unsigned long long n, unique, hit, stale, miss, evicted, evicted_dirty, stale_dirty, flushed;
};

// Small block of device-resident scalars that the kernels of one call hand to each other, so
// that no count has to travel to the host between kernels.
struct DState {
    uint32_t t;          // iteration = number of non-empty lookups; the LRU time stamp
    int32_t size;        // cached rows
    int32_t size_before; // those before the current lookup's fetches
    uint32_t n_unique;   // distinct valid ids of the current call
    uint32_t n_valid;    // ids of the current call that lie in [0, vocab)
    int32_t cut_slot;    // trim, counted beside the fetches: the rows fetched into slots up to this one are victims (-1: none)
    uint32_t err;        // sticky ERRBIT_*
    uint32_t ev_n[2];    // ids recorded by a trim; trims alternate, the lookup in between clears the idle count
    uint32_t sel_take;   // trim: how many of the rows whose policy key equals sel_tau are evicted (in slot order)
    uint32_t sel_tau;    // trim: policy key of the last row to evict
    int32_t over;        // trim: rows above capacity when the select ran (what the eviction removes)
    uint32_t push_n[2];  // host-backed table: rows a trim staged for write-back; trims alternate like ev_n
    uint32_t pf_n[2];    // host-backed table: keys of a coming batch listed for fetching ahead; the lists alternate
    Counters call[2];    // per-call counters: calls alternate between the two, the idle one is cleared meanwhile
    Counters total;
};

__device__ __forceinline__ uint32_t lane_id()
{
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Number of set bits of a 64-lane mask below the calling lane.
__device__ __forceinline__ uint32_t mask_rank(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// A value from another lane of the wave through the data-parallel-primitive path of the vector ALU
// (no trip through the LDS crossbar, as a shuffle makes): lanes that have no source, or are outside
// the row mask, get 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}

// Inclusive scan over the wave: within each row of 16 lanes (shift right by 1, 2, 4, 8), then the
// last lane of rows 0 and 2 into rows 1 and 3, then lane 31 into the upper half.  All lanes active.
// (A shuffle per step is six trips through LDS in a row; every kernel of the step waits for one to
// four such scans: lookups of 53248 ids 71.3 -> 68.0 us, a step of 106496 ids 75.9 -> 73.3 us.)
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xf>(v);
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v), WAVE - 1);
}

// Exclusive scan of one value per thread over a block of NW waves; `total` gets the block sum.
// `lds` needs NW words.  Contains block barriers: call from all threads.
template <int NW>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *lds, uint32_t &total)
{
    const uint32_t lane = lane_id(), w = threadIdx.x / WAVE;
    const uint32_t inc = wave_incl_scan(v);
    __syncthreads();                       // lds may still be read from a previous use
    if (lane == WAVE - 1) lds[w] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) { const uint32_t c = lds[i]; before += (uint32_t)i < w ? c : 0u; all += c; }
    total = all;
    return before + inc - v;
}

// Sum over the block of one value per thread (all threads get it).  `lds` needs NW words.
template <int NW>
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *lds)
{
    const uint32_t lane = lane_id(), w = threadIdx.x / WAVE;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) lds[w] = v;
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) s += lds[i];
    return s;
}

// Sum of a[0 .. count) computed by the whole block (every thread gets it).  Loads go out eight
// at a time per thread before anything is added.
template <int NW>
__device__ __forceinline__ uint32_t block_sum_array(const uint32_t *a, uint32_t count, uint32_t *lds)
{
    uint32_t v = 0;
    for (uint32_t i0 = threadIdx.x; i0 < count; i0 += 8 * NW * WAVE) {
        uint32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) { const uint32_t i = i0 + u * NW * WAVE; x[u] = i < count ? a[i] : 0u; }
#pragma unroll
        for (int u = 0; u < 8; ++u) v += x[u];
    }
    return block_sum<NW>(v, lds);
}

// Row geometry: a row of `dim` floats is handled by a group of `lanes` consecutive lanes
// (power of two, at most 64), each moving VEC floats per step.
struct RowGeom {
    int dim;      // floats per row
    int vec;      // 4 if dim % 4 == 0, else 1
    int lanes;    // lanes per row group
    int chunks;   // dim / vec
};

template <int VEC> struct VecT;
template <> struct VecT<4> { using type = float4; };
template <> struct VecT<1> { using type = float; };

template <int VEC>
__device__ __forceinline__ void row_copy(float *dst, const float *src, int chunks, int lanes, int gl)
{
    using V = typename VecT<VEC>::type;
    const V *s = reinterpret_cast<const V *>(src);
    V *d = reinterpret_cast<V *>(dst);
    for (int c = gl; c < chunks; c += lanes) d[c] = s[c];
}

} // namespace het
