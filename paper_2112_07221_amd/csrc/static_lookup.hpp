// The Read without a cache object (het_lookup_nocache_static): out[i] = table[ids[i]].
//
// Nothing is cached, no gradient follows and nobody asks for the distinct keys, so the ids need no
// order: every position reads its own row, and rows of popular ids come out of the caches.  One
// launch (before: sort, run marking and gather, ten launches).  Small calls are latency only (id, row,
// store): 208 ids of 64 floats took 27 us of kernels and 35 us a call, bound by enqueueing ten
// launches; now 2.5 us (launches in a row) and 8.3 us a call, most of it the caller's Python.
// Large calls are bound by HBM: 65536 ids of 64 floats 7.4 us, 4.5 TB/s of rows read and written.
// One row per row group: four in flight were slower at 4096 x 64 (2.8 against 2.4 us), 32768 x 64 (5.1 /
// 4.6) and 32768 x 256 (12.3 / 11.9) and faster only at the very largest call (65536 x 128: 13.4 / 14.5):
// with this many short workgroups the rows in flight come from the workgroups.
#pragma once
#include "common.hpp"

namespace het {

constexpr uint32_t STATIC_THREADS = 256;
constexpr uint32_t STATIC_CHECK_LOADS = 16;          // ids a thread of the checking workgroup has in flight

// Says whether any id lies outside the vocabulary: one workgroup beside the gather's, so that the
// answer needs neither a counter to be cleared first nor a launch of its own.
__device__ __forceinline__ void static_check_body(const int64_t *__restrict__ ids, uint32_t n, uint32_t vocab, uint32_t *err_bits)
{
    bool bad = false;
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += STATIC_CHECK_LOADS * STATIC_THREADS) {
        int64_t id[STATIC_CHECK_LOADS];
#pragma unroll
        for (uint32_t u = 0; u < STATIC_CHECK_LOADS; ++u) { const uint32_t i = i0 + u * STATIC_THREADS; id[u] = i < n ? ids[i] : 0; }
#pragma unroll
        for (uint32_t u = 0; u < STATIC_CHECK_LOADS; ++u) bad |= id[u] < 0 || id[u] >= (int64_t)vocab;
    }
    const int any = __syncthreads_or(bad);
    if (threadIdx.x == 0) *err_bits = any ? ERRBIT_RANGE : 0u;
}

static __global__ void static_clear_kernel(uint32_t *err_bits) { *err_bits = 0; }

// CHECK: the last workgroup checks the ids; otherwise a workgroup that meets a bad id sets the bit
// itself (err_bits was cleared by a launch before this one).
template <int VEC, bool CHECK>
__global__ __launch_bounds__(STATIC_THREADS) void static_lookup_kernel(const float *__restrict__ table, uint32_t vocab, RowGeom g,
                                                                       const int64_t *__restrict__ ids, uint32_t n, float *__restrict__ out,
                                                                       uint32_t *__restrict__ err_bits)
{
    using V = typename VecT<VEC>::type;
    if (CHECK && blockIdx.x + 1 == gridDim.x) { static_check_body(ids, n, vocab, err_bits); return; }
    const uint32_t i = blockIdx.x * (STATIC_THREADS / g.lanes) + threadIdx.x / g.lanes;
    if (i >= n) return;
    const int gl = threadIdx.x % g.lanes;
    const int64_t id = ids[i];
    const bool ok = id >= 0 && id < (int64_t)vocab;
    const V *row = reinterpret_cast<const V *>(table + (size_t)(ok ? id : 0) * g.dim);
    V *to = reinterpret_cast<V *>(out + (size_t)i * g.dim);
    for (int c = gl; c < g.chunks; c += g.lanes) to[c] = ok ? row[c] : V{};
    if (!CHECK && err_bits && !ok && gl == 0) atomicOr(err_bits, ERRBIT_RANGE);
}

} // namespace het
