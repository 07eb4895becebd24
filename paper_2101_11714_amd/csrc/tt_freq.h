// Access-frequency tracker of the semi-dynamic cache (Section 4.2 of the paper): an
// open-addressing hash table row -> number of accesses, kept on the device and updated from the
// index stream of every step.  Integer only.
//
// An entry is one 64-bit word, (row << 32) | count, empty = all ones: inserting a row is one
// compare-and-swap, counting an access one 64-bit add of the right amount to the same word.
// Equal rows inside a wave are combined first (one add per distinct row and wave), so that a
// row that makes up a fifth of the stream does not turn into as many adds to one address.
#pragma once

#include "tt_common.h"

namespace tt {

constexpr uint64_t FREQ_EMPTY = ~0ull;

struct FreqDev {
    unsigned long long *table;
    unsigned long long *stats;      // [0] distinct rows in the table, [1] accesses dropped because it was full
    uint32_t mask;                  // capacity - 1
};

__global__ __launch_bounds__(WG) void freq_reset_kernel(FreqDev f)
{
    const uint32_t i = blockIdx.x * WG + threadIdx.x;
    if (i <= f.mask) f.table[i] = FREQ_EMPTY;
    if (i < 2) f.stats[i] = 0ull;
}

// add `n` accesses of `row`; linear probing from the same hash as the cache map
__device__ __forceinline__ void freq_add(const FreqDev &f, uint32_t row, uint32_t n)
{
    uint32_t h = cache_hash(row, f.mask);
    for (uint32_t probes = 0; probes <= f.mask; ++probes) {
        unsigned long long e = __hip_atomic_load(&f.table[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (e == FREQ_EMPTY) {
            const unsigned long long fresh = (unsigned long long)row << 32;
            e = atomicCAS(&f.table[h], (unsigned long long)FREQ_EMPTY, fresh);
            if (e == FREQ_EMPTY) {
                atomicAdd(&f.stats[0], 1ull);
                e = fresh;
            }
        }
        if ((uint32_t)(e >> 32) == row) {
            atomicAdd(&f.table[h], (unsigned long long)n);
            return;
        }
        h = (h + 1) & f.mask;
    }
    atomicAdd(&f.stats[1], (unsigned long long)n);                 // table full
}

__global__ __launch_bounds__(WG) void freq_update_kernel(FreqDev f, const int64_t *__restrict__ indices, int L)
{
    const int k = blockIdx.x * WG + threadIdx.x;
    const bool in = k < L;
    const uint32_t my = in ? (uint32_t)indices[k] : 0xFFFFFFFFu;
    const int lane = threadIdx.x & 63;
    // equal rows of the wave are combined without touching memory: the first lane of every
    // distinct row becomes its leader and learns how many lanes hold it ...
    uint64_t rem = __ballot(in);
    uint32_t mine = 0;
    while (rem) {                                                  // uniform: one step per distinct row of the wave
        const int j = __builtin_ctzll(rem);
        const uint32_t rj = (uint32_t)__builtin_amdgcn_readlane((int)my, j);
        const uint64_t m = __ballot(my == rj);
        rem &= ~m;
        if (lane == j) mine = (uint32_t)__popcll(m);
    }
    // ... then all leaders update the table at the same time
    if (mine) freq_add(f, my, mine);
}

// Long streams: a workgroup first counts its FQ_CHUNK positions in a small table in LDS (LDS
// atomics; equal rows meet there), then adds every distinct row of the chunk to the device table
// once.  The hottest row of a Zipf stream then costs one device atomic per chunk, not per wave.
constexpr int FQ_CHUNK = 1024;                   // positions per workgroup
constexpr int FQ_T = 2 * FQ_CHUNK;              // LDS table entries (never full)
constexpr int FQ_NT = 1024;                     // threads

__global__ __launch_bounds__(FQ_NT) void freq_update_chunk_kernel(FreqDev f, const int64_t *__restrict__ indices, int L)
{
    constexpr int NP = FQ_CHUNK / FQ_NT, PER = FQ_T / FQ_NT;
    __shared__ uint32_t lkey[FQ_T], lcnt[FQ_T];
    __shared__ uint32_t s_new, s_lost;
    const int t = threadIdx.x;
    const uint32_t base = blockIdx.x * (uint32_t)FQ_CHUNK, end = (uint32_t)L;
    uint32_t row[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) row[q] = (uint32_t)indices[min(base + q * FQ_NT + t, end - 1)];
    for (int i = t; i < FQ_T; i += FQ_NT) { lkey[i] = 0xFFFFFFFFu; lcnt[i] = 0u; }
    if (t == 0) s_new = s_lost = 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        // (-1, a free entry's key, is no row: as one it would leave its count in a free entry, for whichever row comes there)
        if (base + q * FQ_NT + t >= end || row[q] == 0xFFFFFFFFu) continue;
        uint32_t h = cache_hash(row[q], FQ_T - 1);
        for (;;) {                                                 // ends: at most FQ_CHUNK rows in 2 FQ_CHUNK entries
            const uint32_t old = atomicCAS(&lkey[h], 0xFFFFFFFFu, row[q]);
            if (old == 0xFFFFFFFFu || old == row[q]) { atomicAdd(&lcnt[h], 1u); break; }
            h = (h + 1) & (FQ_T - 1);
        }
    }
    __syncthreads();
    // Every distinct row of the chunk to the device table, all rows of a thread one place further in every round: their loads (and
    // their compare-and-swaps) are in flight together, the adds are not waited for.  What bounds it is that chain of round trips, as long
    // as the longest walk of a wave's rows.  (163,840 positions in a table of 2^20: one entry after the other 33 us; the first places of
    // eight entries of 256 threads together, the walks one after the other 16; so, two entries of 1,024 threads, 10.)
    uint32_t key[PER], h[PER], n[PER], fresh = 0, left = 0;
    unsigned long long e[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        key[q] = lkey[q * FQ_NT + t];
        n[q] = lcnt[q * FQ_NT + t];
        h[q] = cache_hash(key[q], f.mask);
        if (key[q] != 0xFFFFFFFFu) left |= 1u << q;
    }
    for (uint32_t probes = 0; left && probes <= f.mask; ++probes) {
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if ((left >> q) & 1u) e[q] = __hip_atomic_load(&f.table[h[q]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (((left >> q) & 1u) && e[q] == FREQ_EMPTY) {
                const unsigned long long entry = (unsigned long long)key[q] << 32;
                e[q] = atomicCAS(&f.table[h[q]], (unsigned long long)FREQ_EMPTY, entry);
                if (e[q] == FREQ_EMPTY) {
                    e[q] = entry;
                    ++fresh;
                }
            }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (!((left >> q) & 1u)) continue;
            if ((uint32_t)(e[q] >> 32) == key[q]) {
                atomicAdd(&f.table[h[q]], (unsigned long long)n[q]);
                left &= ~(1u << q);
            }
            h[q] = (h[q] + 1) & f.mask;
        }
    }
    if (fresh) atomicAdd(&s_new, fresh);
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if ((left >> q) & 1u) atomicAdd(&s_lost, n[q]);            // table full
    __syncthreads();
    if (t == 0 && s_new) atomicAdd(&f.stats[0], (unsigned long long)s_new);
    if (t == 0 && s_lost) atomicAdd(&f.stats[1], (unsigned long long)s_lost);
}

// rows / counts of the occupied entries, in no particular order; *n_out = how many.  A workgroup compacts FQ_EXPORT
// entries and asks for room once: the adds to *n_out meet at one address (one per wave of 64 entries, 16,384 for a table
// of 2^20, took 198 us; one per 8,192 entries: 7 us, a read of the table).
constexpr int FQ_EXPORT = 32 * WG;

__global__ __launch_bounds__(WG) void freq_export_kernel(FreqDev f, int64_t *__restrict__ rows,
                                                         int64_t *__restrict__ counts, unsigned long long *n_out)
{
    __shared__ int s_tmp[NWAVE + 1];
    __shared__ unsigned long long s_base;
    const int t = threadIdx.x;
    const uint32_t first = blockIdx.x * (uint32_t)FQ_EXPORT + t;
    uint32_t used = 0;
    unsigned long long e[FQ_EXPORT / WG];
#pragma unroll
    for (int q = 0; q < FQ_EXPORT / WG; ++q) {
        const uint32_t i = first + q * WG;
        e[q] = f.table[min(i, f.mask)];
        if (i <= f.mask && e[q] != FREQ_EMPTY) used |= 1u << q;
    }
    int total;
    const int at = block_excl_scan((int)__popc(used), s_tmp, &total);
    if (!total) return;                                            // uniform
    if (t == 0) s_base = atomicAdd(n_out, (unsigned long long)total);
    __syncthreads();
    unsigned long long pos = s_base + (unsigned long long)at;
#pragma unroll
    for (int q = 0; q < FQ_EXPORT / WG; ++q)
        if ((used >> q) & 1u) {
            rows[pos] = (int64_t)(e[q] >> 32);
            counts[pos] = (int64_t)(uint32_t)e[q];
            ++pos;
        }
}

__global__ void freq_zero_kernel(unsigned long long *p) { if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0ull; }

// What a refill puts in place of the old cached set: keys, lines (nr values, 16-byte aligned) and the row -> slot map.  The map is
// built in LDS by the first workgroup and written as a whole while the others copy (IN_LDS), up to CR_MAX_CAPACITY places; a larger
// one is emptied here and filled by cache_insert_kernel.  4,000 rows: emptied, then filled by compare-and-swaps in device memory, a chain
// of round trips per row, 3 + 8 us in two launches; so 6 in one.
constexpr int CR_NT = 1024;
constexpr int64_t CR_MAX_CAPACITY = 16384;       // 128 KB

template <bool IN_LDS>
__global__ __launch_bounds__(CR_NT) void cache_replace_kernel(const int64_t *__restrict__ new_keys, int64_t *__restrict__ keys, int K,
                                                              const float *__restrict__ new_rows, float *__restrict__ rows, int64_t nr,
                                                              uint64_t *__restrict__ table, int64_t capacity)
{
    extern __shared__ __align__(16) unsigned long long cr_map[];              // [capacity]
    const int t = threadIdx.x;
    if (IN_LDS && blockIdx.x == 0) {
        constexpr int NK = 4;                                                 // keys in flight per thread
        const uint32_t mask = (uint32_t)(capacity - 1);
        for (int x = t; x < capacity; x += CR_NT) cr_map[x] = CACHE_EMPTY;
        for (int b = 0; b < K; b += NK * CR_NT) {                             // uniform
            int64_t key[NK];
#pragma unroll
            for (int q = 0; q < NK; ++q) key[q] = new_keys[min(b + q * CR_NT + t, K - 1)];
            __syncthreads();                                                  // (the first time: the map is empty)
#pragma unroll
            for (int q = 0; q < NK; ++q) {
                const int s = b + q * CR_NT + t;
                if (s >= K) continue;
                keys[s] = key[q];
                const unsigned long long entry = ((unsigned long long)(uint32_t)key[q] << 32) | (uint32_t)s;
                uint32_t h = cache_hash((uint32_t)key[q], mask);
                while (atomicCAS(&cr_map[h], (unsigned long long)CACHE_EMPTY, entry) != CACHE_EMPTY) h = (h + 1) & mask;   // ends: capacity >= 2 K
            }
        }
        __syncthreads();
        for (int x = t; x < capacity / 2; x += CR_NT) reinterpret_cast<ulonglong2 *>(table)[x] = reinterpret_cast<const ulonglong2 *>(cr_map)[x];
        return;
    }
    const int64_t wg = (int64_t)blockIdx.x - (IN_LDS ? 1 : 0), wgs = (int64_t)gridDim.x - (IN_LDS ? 1 : 0);
    const int64_t first = wg * CR_NT + t, step = wgs * CR_NT, n4 = nr / 4;
    for (int64_t i = first; i < n4; i += step) reinterpret_cast<float4 *>(rows)[i] = reinterpret_cast<const float4 *>(new_rows)[i];
    for (int64_t i = 4 * n4 + first; i < nr; i += step) rows[i] = new_rows[i];
    if (IN_LDS) return;
    for (int64_t i = first; i < K; i += step) keys[i] = new_keys[i];
    for (int64_t i = first; i < capacity; i += step) table[i] = CACHE_EMPTY;
}

// (rows and table: see cache_replace_kernel)
static inline hipError_t cache_replace(const int64_t *new_keys, int64_t *keys, int K, const float *new_rows, float *rows, int64_t nr, uint64_t *table,
                                       int64_t capacity, hipStream_t st)
{
    const int64_t n4 = nr / 4 + 1, blocks = (n4 + CR_NT - 1) / CR_NT, copy = blocks < 1024 ? blocks : 1024;
    if (capacity <= CR_MAX_CAPACITY && ((uintptr_t)table & 15) == 0) {
        static OncePerDevice once;
        const hipError_t e = allow_dynamic_lds(once, (const void *)cache_replace_kernel<true>, CR_MAX_CAPACITY * 8);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(cache_replace_kernel<true>, dim3((unsigned)copy + 1), dim3(CR_NT), (size_t)capacity * 8, st, new_keys, keys, K, new_rows, rows, nr,
                           table, capacity);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(cache_replace_kernel<false>, dim3((unsigned)copy), dim3(CR_NT), 0, st, new_keys, keys, K, new_rows, rows, nr, table, capacity);
    hipLaunchKernelGGL(cache_insert_kernel, dim3((K + WG - 1) / WG), dim3(WG), 0, st, keys, K, table, (uint32_t)(capacity - 1));
    return hipGetLastError();
}

}  // namespace tt
