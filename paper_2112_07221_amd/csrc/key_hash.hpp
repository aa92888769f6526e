// Find (Algorithm 2 of the paper) where HBM has no room for the direct index (CacheView::slot_of, 4 bytes per
// row of the table): a hash table of the cached keys alone, some 32 to 64 bytes per slot of the cache.
//
// Buckets of 16 entries of 64 bits (id in the high word, slot in the low word, all ones: empty), one bucket to a
// line of 128 bytes.  A key lives in its home bucket or, if that was full when it came, in one of those that
// follow; reach[h] is the largest distance any key of home bucket h was ever displaced, and a search looks at
// buckets h .. h + reach[h] and at nothing else.  A search sees whole buckets, so erasing is writing "empty": no
// tombstones, no rehash.  At most a quarter of the entries are in use.
//
// Searches, inserts and erases have kernels of their own, so that the step's kernels are those of the direct index:
// the search leaves the slots by sorted position, where the probe reads them (CacheView::by_position).  An insert only
// races with inserts (a compare-and-swap on the entry settles it: which entry a key gets depends on that, which slot
// it has does not).  106496 ids, 75758 keys, 64 million rows of 64 floats: 73 us a step with the index in HBM, 87
// with this, 320 with the index in pinned host memory, where every Find crosses the link (and which is left for where
// not even this finds room).
#pragma once
#include "common.hpp"

namespace het {

constexpr int BUCKET_ENTRIES = 16;
constexpr uint64_t ENTRY_EMPTY = ~0ull;

struct KeyHash {
    uint64_t *entries;    // [n_buckets][BUCKET_ENTRIES], or nullptr: the direct index is in use
    uint32_t *reach;      // [n_buckets]
    uint32_t mask;        // n_buckets - 1 (a power of two)
    int shift;            // 64 - log2(n_buckets)
};

__device__ __forceinline__ uint32_t key_home(const KeyHash &h, uint32_t key)
{
    return (uint32_t)(((uint64_t)key * 0x9E3779B97F4A7C15ull) >> 1 >> (h.shift - 1)) & h.mask;      // (in two steps: with one bucket the shift is 64)
}

// The bucket's entries: key in the odd words, slot in the even ones.
struct Bucket { uint4 v[BUCKET_ENTRIES / 2]; };
__device__ __forceinline__ Bucket load_bucket(const KeyHash &h, uint32_t b)
{
    Bucket k;
    const uint4 *line = reinterpret_cast<const uint4 *>(h.entries + (size_t)b * BUCKET_ENTRIES);
#pragma unroll
    for (int q = 0; q < BUCKET_ENTRIES / 2; ++q) k.v[q] = line[q];
    return k;
}

// Slot of `key` or SLOT_NONE, and where its entry is.  (No cached key is KEY_NONE: ids are below 2^32 - 1.)
__device__ __forceinline__ int32_t key_find(const KeyHash &h, uint32_t key, size_t &at)
{
    const uint32_t home = key_home(h, key), reach = h.reach[home];
    for (uint32_t d = 0; d <= reach; ++d) {
        const uint32_t b = (home + d) & h.mask;
        const Bucket k = load_bucket(h, b);
        int32_t slot = SLOT_NONE;
        uint32_t e = 0;
#pragma unroll
        for (int q = 0; q < BUCKET_ENTRIES / 2; ++q) {
            if (k.v[q].y == key) { slot = (int32_t)k.v[q].x; e = 2 * q; }
            if (k.v[q].w == key) { slot = (int32_t)k.v[q].z; e = 2 * q + 1; }
        }
        if (slot != SLOT_NONE) { at = (size_t)b * BUCKET_ENTRIES + e; return slot; }
    }
    return SLOT_NONE;
}

// The slot of the key at every sorted position where the probe asks for one: the head of every run of equal keys and
// each wave's first lane.
static __global__ __launch_bounds__(256) void key_find_kernel(KeyHash h, const uint32_t *__restrict__ skey, uint32_t n, uint32_t vocab, int32_t *__restrict__ found)
{
    const uint32_t j = blockIdx.x * 256u + threadIdx.x;
    if (j >= n) return;
    const uint32_t key = skey[j];
    if (key == vocab || (j % WAVE != 0 && skey[j - 1] == key)) return;
    size_t at;
    found[j] = key_find(h, key, at);
}

// The keys a lookup fetched (none of them is there yet).  cls and head_slot are valid at run heads.
static __global__ __launch_bounds__(256) void key_insert_kernel(KeyHash h, const uint32_t *__restrict__ skey, const uint8_t *__restrict__ cls,
                                                         const int32_t *__restrict__ head_slot, uint32_t n, uint32_t vocab)
{
    const uint32_t j = blockIdx.x * 256u + threadIdx.x;
    if (j >= n) return;
    const uint32_t key = skey[j];
    if (key == vocab || (j > 0 && skey[j - 1] == key) || cls[j] != (uint8_t)CLS_MISS) return;
    const unsigned long long entry = ((unsigned long long)key << 32) | (uint32_t)head_slot[j];
    const uint32_t home = key_home(h, key);
    for (uint32_t d = 0; d <= h.mask; ++d) {             // (ends long before: three quarters of the entries are empty)
        const uint32_t b = (home + d) & h.mask;
        const Bucket k = load_bucket(h, b);
        uint32_t empty = 0;
#pragma unroll
        for (int q = 0; q < BUCKET_ENTRIES / 2; ++q) {
            if (k.v[q].y == KEY_NONE) empty |= 1u << (2 * q);
            if (k.v[q].w == KEY_NONE) empty |= 2u << (2 * q);
        }
        unsigned long long *line = reinterpret_cast<unsigned long long *>(h.entries + (size_t)b * BUCKET_ENTRIES);
        for (; empty; empty &= empty - 1) {
            if (atomicCAS(&line[__ffs(empty) - 1], (unsigned long long)ENTRY_EMPTY, entry) != (unsigned long long)ENTRY_EMPTY) continue;
            if (d) atomicMax(&h.reach[home], d);
            return;
        }
    }
}

// The keys a trim dropped.
static __global__ __launch_bounds__(256) void key_erase_kernel(KeyHash h, const uint32_t *__restrict__ ev_ids, const uint32_t *__restrict__ ev_n)
{
    const uint32_t n = *ev_n;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
        size_t at;
        if (key_find(h, ev_ids[i], at) != SLOT_NONE) h.entries[at] = ENTRY_EMPTY;
    }
}

} // namespace het
