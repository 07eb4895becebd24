// The K smallest of n distinct keys, in order (the cache population of Section 4.2: most used rows first, ties by row
// id; the key is the inverted count above the row id).  A full sort of the candidates orders all of them, eight passes
// over 64-bit keys, for the few thousand that are kept.  Here one histogram over the leading bits of the counts finds the
// class of counts that holds the K-th key; if the keys up to the end of that class are few enough they are compacted and
// ranked by counting the smaller ones, else (thousands of candidates with the count of the K-th) the class is
// narrowed down first, digit by digit.  40 M-row table, 77,000 candidates, K = 4,000: the sort took 104 us in 16
// launches (its passes are chains of memory round trips), this 21 us in 3.
#pragma once

#include "tt_common.h"
#include "tt_sort.h"
#include "tt_rows.h"

namespace tt {

constexpr int TK_BITS = 12, TK_BINS = 1 << TK_BITS;
constexpr int TK_CLASSES = 33 * 64;              // classes of counts (topk_class)
constexpr int TK_NT = 1024, TK_TILE = 4096;      // threads, and keys, per workgroup of a pass
constexpr int TK_MAX_K = 8192;                   // ranking compares every pair: 5 us for 4,000 keys, 20 us for this many
// More candidates than every workgroup should read again for each digit where ties have to be narrowed down.  262,144 candidates, K = 8,192,
// of one count 116 us a refill, of 19 counts 114, counts by a Zipf law 83; sorted, 262,145: 120, 118, 119.
constexpr int TK_MAX_N = 1 << 18;
constexpr int TK_RANK_KEYS = 8;                  // keys a workgroup ranks, 32 threads each

struct TopkState {
    uint32_t count;                              // keys taken
};

struct TopkWs {
    uint64_t *keys, *taken;                      // [n], [TK_MAX_K]
    uint32_t *hist;                              // [tiles][TK_CLASSES]
    TopkState *state;
};

// Everything lies in the workspace of a sort of n keys (n > TK_MAX_K).
static inline TopkWs topk_ws(const SortWs &s, int n)
{
    // tiles TK_CLASSES + 1 <= (n / TK_TILE + 1) TK_CLASSES + 1 <= n: the histograms and the state fit the n payload words
    static_assert(TK_CLASSES < TK_TILE && (int64_t)TK_CLASSES * TK_TILE < (int64_t)TK_MAX_K * (TK_TILE - TK_CLASSES), "room");
    const int tiles = (n + TK_TILE - 1) / TK_TILE;
    return TopkWs{s.k0, s.k1, s.v0, (TopkState *)(s.v0 + tiles * TK_CLASSES)};
}

// key = inverted count (32 bits) above rb bits of the row
__device__ __forceinline__ uint32_t topk_count(int64_t count) { return (uint64_t)count > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)count; }
__device__ __forceinline__ uint64_t topk_key(int64_t row, int64_t count, int rb)
{
    return ((uint64_t)(~topk_count(count)) << rb) | ((uint64_t)row & ((1ull << rb) - 1ull));
}

__global__ __launch_bounds__(WG) void topk_keys_kernel(const int64_t *__restrict__ rows, const int64_t *__restrict__ counts, int n, int rb,
                                                       uint64_t *__restrict__ keys)
{
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i < n) keys[i] = topk_key(rows[i], counts[i], rb);
}

// Class of a count: its number of bits (0..32) and the 6 bits below the leading one, larger counts in smaller classes.
// Counts below 128 are classes of their own; a class is always a set of keys with common leading bits.
__device__ __forceinline__ uint32_t topk_class(uint32_t count)
{
    const int nb = count ? 32 - __clz((int)count) : 0;
    const uint32_t frac = nb > 7 ? (count >> (nb - 7)) & 63u : (count << (7 - nb)) & 63u;
    return (uint32_t)(32 - nb) * 64u + (63u - frac);
}

// Keys, and the histogram of their classes, of a tile of candidates: hist[tile][TK_CLASSES].
__global__ __launch_bounds__(TK_NT) void topk_class_kernel(const int64_t *__restrict__ rows, const int64_t *__restrict__ counts, int n, int rb,
                                                           uint64_t *__restrict__ keys, uint32_t *__restrict__ hist, TopkState *__restrict__ state)
{
    constexpr int PER = TK_TILE / TK_NT;
    __shared__ uint32_t h[TK_CLASSES];
    const int t = threadIdx.x, lane = t & 63, base = blockIdx.x * TK_TILE;
    int64_t r[PER], c[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) { r[q] = rows[min(base + q * TK_NT + t, n - 1)]; c[q] = counts[min(base + q * TK_NT + t, n - 1)]; }
    for (int x = t; x < TK_CLASSES; x += TK_NT) h[x] = 0u;
    if (blockIdx.x == 0 && t == 0) state->count = 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const bool in = base + q * TK_NT + t < n;
        const uint32_t x = topk_class(topk_count(c[q]));
        if (in) keys[base + q * TK_NT + t] = topk_key(r[q], c[q], rb);
        // (most rows have been used once or twice: lanes of one class, that of the first lane, add together)
        const uint64_t same = __ballot(in && x == (uint32_t)__builtin_amdgcn_readfirstlane((int)x));
        if ((same >> lane) & 1) {
            if (!(same & lanemask_lt())) atomicAdd(&h[x], (uint32_t)__popcll(same));
        } else if (in) {
            atomicAdd(&h[x], 1u);
        }
    }
    __syncthreads();
    for (int x = t; x < TK_CLASSES; x += TK_NT) hist[(size_t)blockIdx.x * TK_CLASSES + x] = h[x];
}

// The keys up to the end of the class with the K-th key, in any order.  Every workgroup finds that class itself from all tiles'
// histograms.  Where the keys up to its end are more than can be ranked, it then looks for more leading bits of the K-th key: a histogram of the
// next bits over the keys of the class, as often as needed (all workgroups alike: no slower than one of them, and no launch of its own
// for what is hardly ever needed).
__global__ __launch_bounds__(TK_NT) void topk_take_kernel(const uint64_t *__restrict__ keys, int n, int K, int rb, const uint32_t *__restrict__ hist, TopkState *__restrict__ state, uint64_t *__restrict__ taken)
{
    constexpr int W = TK_NT / WAVE, PER = TK_TILE / TK_NT, NF = 8, CPT = (TK_CLASSES + TK_NT - 1) / TK_NT, BPT = TK_BINS / TK_NT;
    __shared__ uint32_t h[TK_BINS];
    __shared__ int s_tmp[W];
    __shared__ uint64_t s_prefix;
    __shared__ int s_shift;
    __shared__ uint32_t s_before, s_remaining, s_class, s_base;
    const int t = threadIdx.x, tiles = gridDim.x, base = blockIdx.x * TK_TILE;
    uint64_t k[PER];
    {
#pragma unroll
        for (int q = 0; q < PER; ++q) k[q] = keys[min(base + q * TK_NT + t, n - 1)];
        uint32_t v[CPT], sum = 0;
#pragma unroll
        for (int x = 0; x < CPT; ++x) v[x] = 0u;
        if (t * CPT < TK_CLASSES) {
            static_assert(TK_CLASSES % CPT == 0, "whole threads");
            for (int b = 0; b < tiles; b += NF) {
                uint32_t u[NF][CPT];
#pragma unroll
                for (int q = 0; q < NF; ++q)
#pragma unroll
                    for (int x = 0; x < CPT; ++x) u[q][x] = hist[(size_t)min(b + q, tiles - 1) * TK_CLASSES + t * CPT + x];
#pragma unroll
                for (int q = 0; q < NF; ++q)
#pragma unroll
                    for (int x = 0; x < CPT; ++x) v[x] += b + q < tiles ? u[q][x] : 0u;
            }
        }
#pragma unroll
        for (int x = 0; x < CPT; ++x) sum += v[x];
        int total;
        uint32_t before = (uint32_t)rw_scan_of<W>((int)sum, s_tmp, &total);
#pragma unroll
        for (int x = 0; x < CPT; ++x) {
            if (before < (uint32_t)K && (uint32_t)K <= before + v[x]) {      // one thread, one class
                // leading bits of the inverted counts of the class: nb bits of the count, the lower nb - 7 of them open
                const int cl = t * CPT + x, nb = 32 - cl / 64;
                const uint32_t frac = 63u - (uint32_t)(cl % 64);
                const int open = nb > 7 ? nb - 7 : 0;
                const uint64_t top = nb == 0 ? 0ull : (nb > 7 ? 64ull + frac : ((64ull + frac) >> (7 - nb)));   // the count without its open bits
                s_prefix = (0xFFFFFFFFull >> open) - top;
                s_shift = rb + open;
                s_before = before;
                s_remaining = (uint32_t)K - before;
                s_class = v[x];
            }
            before += v[x];
        }
    }
    __syncthreads();
    while (s_before + s_class > TK_MAX_K && s_shift > 0) {                   // uniform; the shift falls in every round
        const int bits = min(TK_BITS, s_shift), shift = s_shift - bits;
        const uint64_t prefix = s_prefix;
        for (int x = t; x < TK_BINS; x += TK_NT) h[x] = 0u;
        __syncthreads();
        for (int b = t; b < n; b += NF * TK_NT) {
            uint64_t x[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) x[q] = keys[min(b + q * TK_NT, n - 1)];
#pragma unroll
            for (int q = 0; q < NF; ++q)
                if (b + q * TK_NT < n && (x[q] >> (shift + bits)) == prefix) atomicAdd(&h[(uint32_t)(x[q] >> shift) & ((1u << bits) - 1u)], 1u);
        }
        __syncthreads();
        uint32_t v[BPT], sum = 0;
#pragma unroll
        for (int q = 0; q < BPT; ++q) { v[q] = h[t * BPT + q]; sum += v[q]; }
        int total;
        uint32_t before = (uint32_t)rw_scan_of<W>((int)sum, s_tmp, &total);
        const uint32_t want = s_remaining, below = s_before;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            if (before < want && want <= before + v[q]) {                    // one thread
                s_prefix = (prefix << bits) | (uint64_t)(t * BPT + q);
                s_shift = shift;
                s_before = below + before;
                s_remaining = want - before;
                s_class = v[q];
            }
            before += v[q];
        }
        __syncthreads();
    }
    const int shift = s_shift;
    const uint64_t prefix = s_prefix;
    int mine = 0;
    uint32_t in = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (base + q * TK_NT + t < n && (k[q] >> shift) <= prefix) { in |= 1u << q; ++mine; }
    int total;
    int at = rw_scan_of<W>(mine, s_tmp, &total);
    if (!total) return;                          // uniform
    if (t == 0) s_base = atomicAdd(&state->count, (uint32_t)total);
    __syncthreads();
    at += (int)s_base;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if ((in >> q) & 1u) {
            if (at < TK_MAX_K) taken[at] = k[q]; // (more only if the candidates are not distinct)
            ++at;
        }
}

// out[rank of a key] = its row, for ranks below K: 32 threads count the smaller ones of m <= TK_MAX_K keys (and the equal
// ones before it, so that keys that are not distinct get ranks of their own all the same)
// m is read from the state where it was found on the device.
__global__ __launch_bounds__(WG) void topk_rank_kernel(const uint64_t *__restrict__ keys, int m, const TopkState *__restrict__ state, int K,
                                                       int rb, int64_t *__restrict__ out)
{
    constexpr int STEP = 4096, PER = WG / TK_RANK_KEYS;
    __shared__ uint64_t s_keys[STEP];
    const int t = threadIdx.x, sub = t % PER, i = (int)blockIdx.x * TK_RANK_KEYS + t / PER;
    if (state) m = (int)min(state->count, (uint32_t)TK_MAX_K);
    if ((int)blockIdx.x * TK_RANK_KEYS >= m) return;                         // uniform
    const uint64_t my = keys[min(i, m - 1)];
    int rank = 0;
    for (int b = 0; b < m; b += STEP) {
        const int c = min(STEP, m - b);
#pragma unroll
        for (int q = 0; q < STEP / WG; ++q) {
            const int x = q * WG + t;
            s_keys[x] = keys[min(b + x, m - 1)];
        }
        __syncthreads();
        const int before = min(max(i - b, 0), c);
        int x = sub;
#pragma unroll 8
        for (; x < before; x += PER) rank += s_keys[x] <= my;
#pragma unroll 8
        for (; x < c; x += PER) rank += s_keys[x] < my;
        __syncthreads();
    }
#pragma unroll
    for (int d = 1; d < PER; d <<= 1) rank += __shfl_xor(rank, d);
    if (sub == 0 && i < m && rank < K) out[rank] = (int64_t)(my & ((1ull << rb) - 1ull));
}

__global__ __launch_bounds__(WG) void take_rows_kernel(const uint64_t *__restrict__ sorted, int K, int rb, int64_t *__restrict__ keys)
{
    const int s = blockIdx.x * WG + threadIdx.x;
    if (s < K) keys[s] = (int64_t)(sorted[s] & ((1ull << rb) - 1ull));
}

// keys[0..K) = the rows of the K most used of n candidates (0 < K <= n), most used first, ties by row id.  s: the
// workspace of a sort of n keys.  Up to TK_MAX_K candidates are ranked directly; beyond K = TK_MAX_K (ranking compares
// pairs) or n = TK_MAX_N (see topk_take_kernel) all candidates are sorted.
static inline hipError_t topk_rows(const SortWs &s, const int64_t *cand_rows, const int64_t *cand_counts, int n, int K, int64_t num_rows,
                                   int64_t *keys, hipStream_t st)
{
    int rb = 1;
    while ((1ll << rb) < num_rows) ++rb;         // rows are below 2^31: 33 to 63 bits in all
    const int blocks = (n + WG - 1) / WG, tiles = (n + TK_TILE - 1) / TK_TILE;
    const bool select = n > TK_MAX_K && K <= TK_MAX_K && n <= TK_MAX_N;
    if (select) {
        const TopkWs w = topk_ws(s, n);
        hipLaunchKernelGGL(topk_class_kernel, dim3(tiles), dim3(TK_NT), 0, st, cand_rows, cand_counts, n, rb, w.keys, w.hist, w.state);
        hipLaunchKernelGGL(topk_take_kernel, dim3(tiles), dim3(TK_NT), 0, st, w.keys, n, K, rb, w.hist, w.state, w.taken);
        hipLaunchKernelGGL(topk_rank_kernel, dim3(TK_MAX_K / TK_RANK_KEYS), dim3(WG), 0, st, w.taken, 0, w.state, K, rb, keys);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(topk_keys_kernel, dim3(blocks), dim3(WG), 0, st, cand_rows, cand_counts, n, rb, s.k0);
    if (n <= TK_MAX_K) {
        hipLaunchKernelGGL(topk_rank_kernel, dim3((n + TK_RANK_KEYS - 1) / TK_RANK_KEYS), dim3(WG), 0, st, s.k0, n, (const TopkState *)nullptr,
                           K, rb, keys);
    } else {
        uint64_t *ks; uint32_t *vs;
        hipError_t e = radix_sort(s, n, 32 + rb, st, &ks, &vs);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(take_rows_kernel, dim3((K + WG - 1) / WG), dim3(WG), 0, st, ks, K, rb, keys);
    }
    return hipGetLastError();
}

}  // namespace tt
