// The K smallest of n distinct keys, in order (the cache population of Section 4.2: most used rows first, ties by row
// id; the key is the inverted count above the row id).  A full sort of the candidates orders all of them, eight passes
// over 64-bit keys, for the few thousand that are kept.  Here one histogram over the leading bits of the counts finds the
// class of counts that holds the K-th key; if the keys up to the end of that class are few enough they are compacted and
// ranked by counting the smaller ones, else (thousands of candidates with the count of the K-th) a single workgroup
// narrows the class down first, digit by digit.  40 M-row table, 77,000 candidates, K = 4,000: the sort took 104 us in 16
// launches (its passes are chains of memory round trips), this 23 us in 5.
#pragma once

#include "tt_common.h"
#include "tt_sort.h"

namespace tt {

constexpr int TK_BITS = 12, TK_BINS = 1 << TK_BITS;
constexpr int TK_TILE = 2048;                    // keys per workgroup of a pass
constexpr int TK_MAX_K = 8192;                   // ranking compares every pair: 5 us for 4,000 keys, 20 us for this many
constexpr int TK_MAX_N = 1 << 18;                // more candidates than a single workgroup should have to narrow down
constexpr int TK_RANK_KEYS = 8;                  // keys a workgroup ranks, 32 threads each
constexpr int TK_NARROW_WG = 1024;

struct TopkState {
    uint64_t prefix;                             // the leading bits of the K-th key found so far ...
    int shift;                                   // ... and how many bits follow
    uint32_t before, remaining;                  // keys below that class, keys still to take inside it
    uint32_t blocks, count;
};

struct TopkWs {
    uint64_t *keys, *taken;                      // [n], [TK_MAX_K]
    uint32_t *hist;                              // [TK_BINS]
    TopkState *state;
};

// Everything lies in the workspace of a sort of n keys (n > TK_MAX_K).
static inline TopkWs topk_ws(const SortWs &s)
{
    static_assert(TK_MAX_K >= TK_BINS + 64, "the histogram and the state fit the n payload words");
    return TopkWs{s.k0, s.k1, s.v0, (TopkState *)(s.v0 + TK_BINS)};
}

// key = inverted count (32 bits) above rb bits of the row; the first workgroup also clears the histogram and the state
__global__ __launch_bounds__(WG) void topk_keys_kernel(const int64_t *__restrict__ rows, const int64_t *__restrict__ counts, int n,
                                                       int rb, uint64_t *__restrict__ keys, uint32_t *__restrict__ hist,
                                                       TopkState *__restrict__ state, int K)
{
    const int i = blockIdx.x * WG + threadIdx.x;
    if (hist && blockIdx.x == 0) {
        for (int x = threadIdx.x; x < TK_BINS; x += WG) hist[x] = 0u;
        if (threadIdx.x == 0) *state = TopkState{0ull, 0, 0u, (uint32_t)K, 0u, 0u};
    }
    if (i >= n) return;
    const uint64_t c = (uint64_t)counts[i];
    const uint32_t inv = 0xFFFFFFFFu - (uint32_t)(c > 0xFFFFFFFFull ? 0xFFFFFFFFull : c);
    keys[i] = ((uint64_t)inv << rb) | ((uint64_t)rows[i] & ((1ull << rb) - 1ull));
}

// Class of a count: its number of bits (0..32) and the 6 bits below the leading one, larger counts in smaller classes.
// Counts below 128 are classes of their own; a class is always a set of keys with common leading bits.
__device__ __forceinline__ uint32_t topk_class(uint32_t count)
{
    const int nb = count ? 32 - __clz((int)count) : 0;
    const uint32_t frac = nb > 7 ? (count >> (nb - 7)) & 63u : (count << (7 - nb)) & 63u;
    return (uint32_t)(32 - nb) * 64u + (63u - frac);
}

// Histogram of the classes; the workgroup that is done last picks the class with the K-th key.
__global__ __launch_bounds__(WG) void topk_class_kernel(const uint64_t *__restrict__ keys, int n, int rb, uint32_t *__restrict__ hist,
                                                        TopkState *__restrict__ state)
{
    constexpr int NB = 33 * 64, PER = (NB + WG - 1) / WG;
    static_assert(NB <= TK_BINS, "the classes fit the histogram");
    __shared__ uint32_t h[NB];
    __shared__ int s_last;
    __shared__ int s_tmp[NWAVE + 1];
    const int t = threadIdx.x;
    uint64_t k[TK_TILE / WG];
#pragma unroll
    for (int q = 0; q < TK_TILE / WG; ++q) k[q] = keys[min((int)blockIdx.x * TK_TILE + q * WG + t, n - 1)];
    for (int x = t; x < NB; x += WG) h[x] = 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TK_TILE / WG; ++q)
        if ((int)blockIdx.x * TK_TILE + q * WG + t < n) atomicAdd(&h[topk_class(~(uint32_t)(k[q] >> rb))], 1u);
    __syncthreads();
    for (int x = t; x < NB; x += WG)
        if (h[x]) atomicAdd(&hist[x], h[x]);
    // This workgroup's adds have to be performed before it counts itself as done.  A barrier alone does not wait for them; they
    // and the loads below go to the point where the whole device meets, so that no fence has to write the caches back.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) s_last = atomicAdd(&state->blocks, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    const uint32_t want = state->remaining;      // 1 <= want <= total; read by everyone before the scan's barriers, written after them
    uint32_t v[PER];
    int sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int x = t * PER + q;
        v[q] = x < NB ? __hip_atomic_load(&hist[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        sum += (int)v[q];
    }
    int total;
    uint32_t before = (uint32_t)block_excl_scan(sum, s_tmp, &total);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (before < want && want <= before + v[q]) {                        // one thread, one class
            // leading bits of the inverted counts of the class: nb bits of the count, the lower nb - 7 of them open
            const int x = t * PER + q, nb = 32 - x / 64;
            const uint32_t frac = 63u - (uint32_t)(x % 64);
            const int open = nb > 7 ? nb - 7 : 0;
            const uint64_t top = nb == 0 ? 0ull : (nb > 7 ? 64ull + frac : ((64ull + frac) >> (7 - nb)));   // the count without its open bits
            state->prefix = (0xFFFFFFFFull >> open) - top;
            state->shift = rb + open;
            state->before = before;
            state->remaining = want - before;
            state->count = 0u;
            state->blocks = v[q];                                            // keys in the class
        }
        before += v[q];
    }
}

// Where the keys up to the end of the class are more than can be ranked, one workgroup finds more leading bits of the
// K-th key: a histogram of the next bits over the keys of the class, as often as needed.
__global__ __launch_bounds__(TK_NARROW_WG) void topk_narrow_kernel(const uint64_t *__restrict__ keys, int n, TopkState *__restrict__ state)
{
    constexpr int W = TK_NARROW_WG / WAVE, PER = TK_BINS / TK_NARROW_WG, NF = 8;
    __shared__ uint32_t h[TK_BINS];
    __shared__ uint32_t s_wave[W];
    __shared__ TopkState s;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (t == 0) s = *state;
    __syncthreads();
    while (s.before + s.blocks > TK_MAX_K && s.shift > 0) {                  // uniform; the shift falls in every round
        const int bits = min(TK_BITS, s.shift), shift = s.shift - bits;
        const uint64_t prefix = s.prefix;
        for (int x = t; x < TK_BINS; x += TK_NARROW_WG) h[x] = 0u;
        __syncthreads();
        for (int b = t; b < n; b += NF * TK_NARROW_WG) {
            uint64_t k[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) k[q] = keys[min(b + q * TK_NARROW_WG, n - 1)];
#pragma unroll
            for (int q = 0; q < NF; ++q)
                if (b + q * TK_NARROW_WG < n && (k[q] >> (shift + bits)) == prefix) atomicAdd(&h[(uint32_t)(k[q] >> shift) & ((1u << bits) - 1u)], 1u);
        }
        __syncthreads();
        uint32_t v[PER], sum = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) { v[q] = h[t * PER + q]; sum += v[q]; }
        uint32_t inc = sum;
#pragma unroll
        for (int d = 1; d < WAVE; d <<= 1) {
            const uint32_t o = __shfl_up(inc, d);
            if (lane >= d) inc += o;
        }
        if (lane == 63) s_wave[w] = inc;
        __syncthreads();
        uint32_t before = inc - sum;
        for (int q = 0; q < w; ++q) before += s_wave[q];
        const uint32_t want = s.remaining, below = s.before;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (before < want && want <= before + v[q]) {                    // one thread
                s.prefix = (prefix << bits) | (uint64_t)(t * PER + q);
                s.shift = shift;
                s.before = below + before;
                s.remaining = want - before;
                s.blocks = v[q];
            }
            before += v[q];
        }
        __syncthreads();
    }
    if (t == 0) *state = s;
}

// the keys up to the end of the class, in any order
__global__ __launch_bounds__(WG) void topk_take_kernel(const uint64_t *__restrict__ keys, int n, TopkState *__restrict__ state,
                                                       uint64_t *__restrict__ taken)
{
    __shared__ int s_tmp[NWAVE + 1];
    __shared__ uint32_t s_base;
    const int t = threadIdx.x, shift = state->shift;
    const uint64_t prefix = state->prefix;
    uint64_t k[TK_TILE / WG];
    int mine = 0;
    uint32_t in = 0;
#pragma unroll
    for (int q = 0; q < TK_TILE / WG; ++q) k[q] = keys[min((int)blockIdx.x * TK_TILE + q * WG + t, n - 1)];
#pragma unroll
    for (int q = 0; q < TK_TILE / WG; ++q)
        if ((int)blockIdx.x * TK_TILE + q * WG + t < n && (k[q] >> shift) <= prefix) { in |= 1u << q; ++mine; }
    int total;
    int at = block_excl_scan(mine, s_tmp, &total);
    if (!total) return;                          // uniform
    if (t == 0) s_base = atomicAdd(&state->count, (uint32_t)total);
    __syncthreads();
    at += (int)s_base;
#pragma unroll
    for (int q = 0; q < TK_TILE / WG; ++q)
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
// pairs) or n = TK_MAX_N (see topk_narrow_kernel) all candidates are sorted.
static inline hipError_t topk_rows(const SortWs &s, const int64_t *cand_rows, const int64_t *cand_counts, int n, int K, int64_t num_rows,
                                   int64_t *keys, hipStream_t st)
{
    int rb = 1;
    while ((1ll << rb) < num_rows) ++rb;         // rows are below 2^31: 33 to 63 bits in all
    const int blocks = (n + WG - 1) / WG, tiles = (n + TK_TILE - 1) / TK_TILE;
    const bool select = n > TK_MAX_K && K <= TK_MAX_K && n <= TK_MAX_N;
    const TopkWs w = topk_ws(s);
    hipLaunchKernelGGL(topk_keys_kernel, dim3(blocks), dim3(WG), 0, st, cand_rows, cand_counts, n, rb, s.k0, select ? w.hist : nullptr,
                       w.state, K);
    if (n <= TK_MAX_K) {
        hipLaunchKernelGGL(topk_rank_kernel, dim3((n + TK_RANK_KEYS - 1) / TK_RANK_KEYS), dim3(WG), 0, st, s.k0, n, (const TopkState *)nullptr,
                           K, rb, keys);
    } else if (select) {
        hipLaunchKernelGGL(topk_class_kernel, dim3(tiles), dim3(WG), 0, st, w.keys, n, rb, w.hist, w.state);
        hipLaunchKernelGGL(topk_narrow_kernel, dim3(1), dim3(TK_NARROW_WG), 0, st, w.keys, n, w.state);
        hipLaunchKernelGGL(topk_take_kernel, dim3(tiles), dim3(WG), 0, st, w.keys, n, w.state, w.taken);
        hipLaunchKernelGGL(topk_rank_kernel, dim3(TK_MAX_K / TK_RANK_KEYS), dim3(WG), 0, st, w.taken, 0, w.state, K, rb, keys);
    } else {
        uint64_t *ks; uint32_t *vs;
        hipError_t e = radix_sort(s, n, 32 + rb, st, &ks, &vs);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(take_rows_kernel, dim3((K + WG - 1) / WG), dim3(WG), 0, st, ks, K, rb, keys);
    }
    return hipGetLastError();
}

}  // namespace tt
