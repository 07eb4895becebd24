// Long index streams with a kept T0: grouping by distinct row, and what works from it.
//
// The positions of a long stream repeat: of 204,800 Zipf-distributed lookups of the Kaggle-shaped table 70,000 are
// distinct, of 8,192 of the Terabyte-shaped one 3,600.  Both passes are linear per row, so the products of Eq. 3 and Eq. 4
// are needed once per distinct row: the forward pass computes a row once and hands it to its positions, the backward pass
// adds up the upstream gradients of a row's positions first.  (Working position by position, the three product kernels
// of that step took 118, 164 and 115 us.)
//
// Pre-pass (index only, five launches; the host never learns how many rows there are):
//   rw_count / rw_scatter   positions grouped by their second digit: one stable counting pass over m2 bins
//   rw_group                a slice's positions in windows of up to RW_WIN: equal rows of a window are found in an LDS hash
//                           table and numbered in the order of their first positions; the window's positions are put in
//                           the order of those numbers.  A row in two windows counts as two: the passes are linear.
//   rw_scan, rw_lists       the distinct rows grouped by first and by third digit (counts per window, column sums, places),
//                           and the table of tiles: up to TP distinct rows of one slice of the second core
// With a cache, positions of cached rows go to RW_CBINS further bins, by their slots; there a window's distinct rows are its
// slots, and `cu` says which u a slot has in it.  Such rows have no tiles and are in no list: the forward pass reads the cache's
// line instead, and in the backward pass a slot's gradient is the sum over the windows of its bin.
// A distinct row is known by its index u = (first place of its window) + (number); places of a window past its distinct
// rows stay unused, so that no count has to travel to the host.
// Everything is stable, so every sum below has a fixed order and results repeat bit for bit.
#pragma once

#include <type_traits>

#include "tt_common.h"
#include "tt_fast.h"
#include "tt_fast_bwd.h"
#include "tt_sort.h"

namespace tt {

constexpr int RW_WIN = 2048;                     // positions of a window, at most (see rw_win)
constexpr int RW_T = 512, RW_NW = RW_T / WAVE;   // threads / waves of the window kernels
constexpr int RW_TILE = 2048, RW_TILE_SHORT = 512;   // positions per workgroup of the counting pass (see rw_tile)
constexpr int RW_PER = 2;                        // positions per thread of it
constexpr int RW_HASH = 4096;
constexpr int RW_MAX_M2 = 1024;                  // bins of the counting pass, those of cached positions among them
constexpr int RW_MAX_M13 = 4096;                 // slices of the first and third core together
constexpr int RW_OFF = 512;                      // samples of the offsets array kept in LDS
constexpr int RW_PIECE = 512;                    // distinct rows per workgroup of the final sums, at most (see rw_piece)

constexpr int RW_CBINS = 128, RW_CSLOTS = 64;    // bins of cached positions (slot modulo RW_CBINS); slots of a bin, at most
constexpr int RW_CWIN = 512;                     // positions of a window of such a bin

struct RowsWs {
    int nb, spb;         // bins of cached positions (0: no cache), slots per bin
    int *cu;             // [windows][spb] u of a bin's slots in a window, -1: none
    int *cwin;           // [nb + 1] first window of every bin
    uint32_t *hist;      // [tiles of the counting pass][m2 + nb rounded up to 4]
    uint32_t *lk, *lrow; // [L] positions and their rows grouped by second digit, cached ones after them by bin
    int *goff;           // [m2 + nb + 1] bounds of those groups
    int *inv;            // [L] position -> u; ~slot of a cached row
    int2 *gkb;           // [L] {position, bag}: the positions of a row are neighbours
    int *gu;             // [L] u of the same places
    int4 *rec;           // [L] by u: {first digit, third digit, first place in gkb, positions} (positions = 0: unused); a slot: {slot, -1, ..}
    int *wd, *wfirst, *wslice;   // [windows] distinct rows, first place, slice (m2 + bin)
    uint32_t *hist2;     // [windows][m1 + m3] distinct rows per slice, then those of earlier windows
    uint32_t *tot2;      // [m1 + m3]
    int *off13;          // [m1 + m3 + 1] bounds of the slices in l13
    int2 *l13;           // [2 L] {u, its first position}, by first digit, then by third digit
    int4 *tiles;         // {slice of the second core, first u, rows, 0}
    int *tile_base;      // [m2 + 1] first tile of every slice
    int *nwin;           // [1] windows in use
    uint32_t *arrived;   // [m1 + m3] workgroups of the final sums that have left a partial sum
    float *rows;         // [L][N] by u: rows of the forward pass
    float *dym;          // [L][N] by u: summed upstream gradients
    float *pbuf;         // [L][sA] by u: G1 gradients
    float *part2;        // [m2 + workgroups of the tile kernel][sB] parts of the second core's gradients
    float *part13;       // [pieces][row] partial sums of slices of more than one piece
    size_t bytes;
};

static inline bool rw_supported(const Params &p)
{
    const int cfg = fast_config(p);
    return cfg >= 2 && cfg <= 5 && p.m2 <= RW_MAX_M2 && p.m1 + p.m3 <= RW_MAX_M13;
}

// Caches that the passes take.
static inline bool rw_cache_supported(const Params &p, int64_t K) { return !K || (K <= RW_CBINS * RW_CSLOTS && p.m2 + RW_CBINS <= RW_MAX_M2); }

// Positions per window.  Longer windows merge more; shorter ones cut a hot row's positions into pieces that different
// workgroups handle, which is what short streams need (8,192 positions, a hot row of 740: one workgroup added these up
// for 13 us).  Up to 262,143 positions half of the longest: a hot row's 2,000 positions are one workgroup's in the forward pass and
// in the sums of the gradients, and that one is the last to finish; longer streams have enough other work and repeat more.  Step, windows of
// 2,048 / 1,024, Zipf-distributed and (uniform) rows: 70,000 positions (2,2,4) rank 64 137 / 121.5 us (188 / 188), rank 32 94 / 93 (101 / 101),
// (4,4,4) rank 64 258 / 237 (508 / 507.5), rank 32 138 / 128 (189.5 / 190); 200,000 192 / 188 (361.6 / 360.4), 125 / 117 (175 / 175),
// 501 / 484 (1,257 / 1,255), 252 / 236 (470 / 471), with a cache 139 / 140; of 512 204 us at rank 64, 204,800 positions.  The two cross later, by
// shape and rank: 270,000 227.6 / 229, 138 / 132, 679 / 668.5, 314 / 302; 400,000 311 / 313, 171 / 170 (365 / 359), 870.5 / 862, 437 / 419
// (939 / 945); 600,000 434 / 457, 277 / 277, 1,231 / 1,313, 603 / 613.  The line is below all of these.
constexpr int64_t RW_LONG_MIN_L = 65536, RW_LONGEST_MIN_L = 262144;
static inline int rw_win(int64_t L) { return L < RW_LONG_MIN_L ? 256 : L < RW_LONGEST_MIN_L ? RW_WIN / 2 : RW_WIN; }
static inline int rw_windows_of(const Params &p, int64_t L, int win) { return (int)(L / win) + p.m2; }
static inline int rw_windows(const Params &p, int64_t L, int64_t K)
{
    return K ? rw_windows_of(p, L, rw_win(L) < RW_CWIN ? rw_win(L) : RW_CWIN) + RW_CBINS : rw_windows_of(p, L, rw_win(L));
}
static inline int rw_tiles(const Params &p, int64_t L, int64_t K, int tp) { return (int)(L / tp) + rw_windows(p, L, K); }
// Distinct rows per workgroup of the final sums: fewer where a table has few slices, so that the sums still spread over the
// device (step of 34,000 positions, (4,4,4) at rank 32, 40 slices per core, uniform rows: 214 us with 512 throughout, 155 so).
static inline int rw_piece(const Params &p, int64_t L)
{
    int n = RW_PIECE;
    while (n > 64 && p.m1 + p.m3 + 2 * (L / n) < 512) n >>= 1;
    return n;
}
// pieces beyond the first one of their slices, at most
static inline int rw_extra(const Params &p, int64_t L) { return (int)(2 * (L / rw_piece(p, L))); }
// room for partial sums: never less for a longer stream (there are fewer than 1,024 extra pieces of less than RW_PIECE rows)
static inline int rw_pieces(const Params &p, int64_t L)
{
    const int64_t small = 2 * (L / 64) < 1024 ? 2 * (L / 64) : 1024, whole = 2 * (L / RW_PIECE);
    return (int)(small > whole ? small : whole) + p.m1 + p.m3;
}
// Positions per workgroup of the counting pass, two per thread: a wave's rounds are one chain of LDS round trips (163,840
// positions, a cache of 1,000 rows to probe: eight of them in 256 threads 13.7 us counting and 12.8 placing, two in 1,024 threads 7.0
// and 11; 8,192 without a cache, 2,048 in 256 threads 9.8 us placing, 512 6.3; 73,000 10 and 7.5); with more workgroups every one
// of them has more counts to read.  Beside a step that does not wait for them the two are alike (8,192 positions 91.8 us either
// way, 6,500 85.9 with 512 / 86.6, 60,000 134.2 / 133.9): the shorter tiles are for the steps and forward passes that do wait.
static inline int rw_tile(int64_t L) { return L < RW_LONG_MIN_L ? RW_TILE_SHORT : RW_TILE; }
static inline int rw_hist_blocks(int64_t L) { return (int)((L + rw_tile(L) - 1) / rw_tile(L)); }

// tile_wgs: workgroups of the tile kernel
static inline RowsWs rw_ws_layout(void *ws, const Params &p, int64_t L, int64_t K, int tile_wgs)
{
    RowsWs w{};
    char *base = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *q = base ? base + off : nullptr; off += align256(bytes); return q; };
    const size_t n = L > 0 ? (size_t)L : 1, nw = (size_t)rw_windows(p, L, K), m13 = (size_t)p.m1 + p.m3;
    w.nb = K ? RW_CBINS : 0;
    w.spb = (int)((K + RW_CBINS - 1) / RW_CBINS);
    w.hist = (uint32_t *)take((size_t)rw_hist_blocks((int64_t)n) * ((p.m2 + w.nb + 3) & ~3) * 4);
    w.lk = (uint32_t *)take(n * 4);
    w.lrow = (uint32_t *)take(n * 4);
    w.goff = (int *)take(((size_t)p.m2 + w.nb + 1) * 4);
    w.inv = (int *)take(n * 4);
    w.gkb = (int2 *)take(n * 8);
    w.gu = (int *)take(n * 4);
    w.rec = (int4 *)take(n * 16);
    w.wd = (int *)take(nw * 4);
    w.wfirst = (int *)take(nw * 4);
    w.wslice = (int *)take(nw * 4);
    w.hist2 = (uint32_t *)take(nw * m13 * 4);
    w.tot2 = (uint32_t *)take(m13 * 4);
    w.off13 = (int *)take((m13 + 1) * 4);
    w.l13 = (int2 *)take(2 * n * 8);
    w.tiles = (int4 *)take((size_t)rw_tiles(p, L, K, 16) * 16);
    w.tile_base = (int *)take(((size_t)p.m2 + 1) * 4);
    w.nwin = (int *)take(4);
    w.arrived = (uint32_t *)take(m13 * 4);
    w.rows = (float *)take(n * p.N * 4);
    w.dym = (float *)take(n * p.N * 4);
    w.pbuf = (float *)take(n * p.sA * 4);
    w.part2 = (float *)take(((size_t)p.m2 + tile_wgs) * p.sB * 4);
    w.part13 = (float *)take((size_t)rw_pieces(p, L) * (p.sA > p.sC ? p.sA : p.sC) * 4);
    w.cu = (int *)take(nw * w.spb * 4);
    w.cwin = (int *)take(K ? ((size_t)w.nb + 1) * 4 : 0);
    w.bytes = off;
    return w;
}

// ---- pre-pass --------------------------------------------------------------------------------------------------------

// the bin of a position: the second digit of its row, or that of a cached row's slot (mark: what rw_count_kernel left in inv)
template <bool CACHED>
__device__ __forceinline__ int rw_bin(const Params &p, uint32_t row, int mark)
{
    return CACHED && mark < 0 ? p.m2 + (~mark & (RW_CBINS - 1)) : (int)select_digit_f64(p, 1, (double)row);
}
static_assert((RW_CBINS & (RW_CBINS - 1)) == 0, "slots are spread over the bins by their low bits");

// bins of a tile of positions, and how many of each; with a cache, inv[k] = ~slot of a cached row, else 0
template <int TILE, bool CACHED>
__global__ __launch_bounds__(TILE / RW_PER) void rw_count_kernel(Params p, const int64_t *__restrict__ indices, int L, CacheDev cache, RowsWs ws)
{
    constexpr int NR = RW_PER, NT = TILE / NR;
    __shared__ uint32_t h[RW_MAX_M2];
    const int t = threadIdx.x, m2p = (p.m2 + (CACHED ? RW_CBINS : 0) + 3) & ~3, base = blockIdx.x * TILE;
    uint32_t row[NR];
    int mark[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        row[q] = (uint32_t)indices[min(base + q * NT + t, L - 1)];
        mark[q] = 0;
    }
    for (int x = t; x < m2p; x += NT) h[x] = 0u;
    if (ws.arrived)
        for (int x = blockIdx.x * NT + t; x < p.m1 + p.m3; x += gridDim.x * NT) ws.arrived[x] = 0u;
    if constexpr (CACHED) {
        uint64_t e[NR];                                            // (the first looks at the table side by side)
#pragma unroll
        for (int q = 0; q < NR; ++q) e[q] = cache.table[cache_hash(row[q], cache.mask)];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            uint32_t at = cache_hash(row[q], cache.mask);
            while (e[q] != CACHE_EMPTY && (uint32_t)(e[q] >> 32) != row[q]) {   // ends: the table is never full
                at = (at + 1) & cache.mask;
                e[q] = cache.table[at];
            }
            if (e[q] != CACHE_EMPTY) mark[q] = ~(int)(uint32_t)e[q];
            if (base + q * NT + t < L) ws.inv[base + q * NT + t] = mark[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NR; ++q)
        if (base + q * NT + t < L) atomicAdd(&h[rw_bin<CACHED>(p, row[q], mark[q])], 1u);
    __syncthreads();
    for (int x = t; x < m2p; x += NT) ws.hist[(size_t)blockIdx.x * m2p + x] = h[x];
}

// exclusive scan of one int per thread over NW waves; tmp: NW ints
template <int NW>
__device__ __forceinline__ int rw_scan_of(int v, int *tmp, int *total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    __syncthreads();
    if (lane == 63) tmp[w] = inc;
    __syncthreads();
    int at = inc - v, all = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        const int x = tmp[q];
        if (q < w) at += x;
        all += x;
    }
    *total = all;
    return at;
}

// Stable placement by second digit.  Every workgroup derives its own starting places from the counts of all tiles (a few
// independent 16-byte loads per thread); wave w ranks its consecutive positions round by round.
template <int TILE, bool CACHED>
__global__ __launch_bounds__(TILE / RW_PER) void rw_scatter_kernel(Params p, const int64_t *__restrict__ indices, int L, int nblk, int bits, RowsWs ws)
{
    constexpr int NR = RW_PER, NT = TILE / NR, NW = NT / WAVE, BPT = RW_MAX_M2 / NT;     // bins per thread: neighbouring ones
    static_assert(NW * RW_MAX_M2 >= 4 * RW_MAX_M2 && BPT >= 1 && BPT <= 4, "room for the partial sums; whole bins per thread");
    __shared__ __align__(16) uint32_t s_cnt[NW][RW_MAX_M2];         // first the partial sums of the counts
    __shared__ uint32_t s_start[RW_MAX_M2];
    __shared__ int s_tmp[NW];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, nbin = p.m2 + (CACHED ? RW_CBINS : 0), m2p = (nbin + 3) & ~3, base = blockIdx.x * TILE + w * (TILE / NW);
    uint32_t row[NR];
    int mark[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        row[q] = (uint32_t)indices[min(base + q * WAVE + lane, L - 1)];
        mark[q] = CACHED ? ws.inv[min(base + q * WAVE + lane, L - 1)] : 0;
    }
    {
        const int q4 = m2p >> 2, most = NW / 4 * 2 * RW_MAX_M2 / m2p, all = NT / q4, nrg = all < most ? all : most, c = t % q4, rg = t / q4;   // q4 <= 256
        uint4 t4 = make_uint4(0u, 0u, 0u, 0u), p4 = t4;
        if (rg < nrg) {
            const uint4 *h4 = reinterpret_cast<const uint4 *>(ws.hist);
            for (int b0 = rg; b0 < nblk; b0 += 16 * nrg) {         // 16 loads in flight (clamped, so none is conditional)
                uint4 v[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = h4[(size_t)min(b0 + q * nrg, nblk - 1) * q4 + c];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int b = b0 + q * nrg;
                    const uint32_t in = b < nblk ? 0xffffffffu : 0u, m = b < (int)blockIdx.x ? 0xffffffffu : 0u;
                    t4.x += v[q].x & in; t4.y += v[q].y & in; t4.z += v[q].z & in; t4.w += v[q].w & in;
                    p4.x += v[q].x & m; p4.y += v[q].y & m; p4.z += v[q].z & m; p4.w += v[q].w & m;
                }
            }
        }
        uint32_t *ptot = &s_cnt[0][0], *ppre = ptot + NW / 2 * RW_MAX_M2;    // [row group][bin] each: nrg m2p fit a half
        if (rg < nrg) {
            *reinterpret_cast<uint4 *>(&ptot[rg * m2p + 4 * c]) = t4;
            *reinterpret_cast<uint4 *>(&ppre[rg * m2p + 4 * c]) = p4;
        }
        __syncthreads();
        uint32_t tot[BPT], pre[BPT], sum = 0;
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            const int bin = BPT * t + q;
            tot[q] = pre[q] = 0u;
            if (bin < m2p)
                for (int g = 0; g < nrg; ++g) { tot[q] += ptot[g * m2p + bin]; pre[q] += ppre[g * m2p + bin]; }
            sum += tot[q];
        }
        int total;
        uint32_t before = (uint32_t)rw_scan_of<NW>((int)sum, s_tmp, &total);
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            const int bin = BPT * t + q;
            if (bin < m2p) {
                s_start[bin] = before + pre[q];
                if (blockIdx.x == 0 && bin <= nbin) ws.goff[bin] = (int)before;
            }
            before += tot[q];
        }
        if (blockIdx.x == 0 && t == 0) ws.goff[nbin] = L;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; ++q)
        for (int bin = t; bin < m2p; bin += NT) s_cnt[q][bin] = 0u;
    __syncthreads();
    int dg[NR], rank[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const bool in = base + q * WAVE + lane < L;
        dg[q] = rw_bin<CACHED>(p, row[q], mark[q]);
        uint64_t same = __ballot(in);
        for (int b = 0; b < bits; ++b) {                           // uniform
            const uint64_t bal = __ballot((dg[q] >> b) & 1);
            same &= (dg[q] >> b) & 1 ? bal : ~bal;
        }
        rank[q] = 0;
        if (in) {
            const uint32_t old = s_cnt[w][dg[q]];
            const int r = (int)__popcll(same & lanemask_lt());
            rank[q] = (int)old + r;
            __builtin_amdgcn_wave_barrier();
            if (r == 0) s_cnt[w][dg[q]] = old + (uint32_t)__popcll(same);
        }
        __builtin_amdgcn_wave_barrier();                           // (LDS of one wave is in order: only the compiler has to keep it)
    }
    __syncthreads();
    for (int bin = t; bin < nbin; bin += NT) {
        uint32_t at = s_start[bin];
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const uint32_t c = s_cnt[q][bin];
            s_cnt[q][bin] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const int k = base + q * WAVE + lane;
        if (k < L) {
            const uint32_t at = s_cnt[w][dg[q]] + (uint32_t)rank[q];
            ws.lk[at] = (uint32_t)k;
            ws.lrow[at] = row[q];
        }
    }
}

// the same over the RW_T threads of the window kernels; tmp: RW_NW ints
__device__ __forceinline__ int rw_scan(int v, int *tmp, int *total) { return rw_scan_of<RW_NW>(v, tmp, total); }

// Which window a workgroup has: its slice and its number in the slice, in s_win (to be read after a barrier); false if there
// is none.
__device__ __forceinline__ bool rw_find_window(const Params &p, int win, const RowsWs &ws, int *s_tmp, int *s_win)
{
    constexpr int PER = RW_MAX_M2 / RW_T;                          // bins per thread
    const int t = threadIdx.x;
    int nwin[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int s = PER * t + q;
        const int n = s < p.m2 ? win : min(win, RW_CWIN);
        nwin[q] = s < p.m2 + ws.nb ? (ws.goff[s + 1] - ws.goff[s] + n - 1) / n : 0;
        sum += nwin[q];
    }
    int total;
    int at = rw_scan(sum, s_tmp, &total);
    if (t == 0 && blockIdx.x == 0) *ws.nwin = total;
    if ((int)blockIdx.x >= total) return false;                    // uniform
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if ((int)blockIdx.x >= at && (int)blockIdx.x < at + nwin[q]) { s_win[0] = PER * t + q; s_win[1] = blockIdx.x - at; }
        at += nwin[q];
    }
    return true;
}

// One window of one slice's positions (win of them, at most): see the file comment.  CACHED, here and below: streams without a
// cache have kernels of their own, without what cached rows need (with it the step of 8,192 positions at rank 64, which has none,
// took 91.8 us instead of 91.1: 0.4 us of grouping, 0.3 of the lists, which waited for wslice, 0.4 of rw_sum_kernel).
//
// All its LDS is dynamic: with 52 KB that the compiler knows of it takes six waves per SIMD to be the most there can be and claims as
// many registers as six leave room for, 80 instead of 48, and then not one workgroup fits beside the tile kernel's at rank 64 (400 of 512
// registers), so that the whole rest of the pre-pass waits for that kernel to end.  100 positions per bag, (2,2,4) rank 64: its 320 workgroups
// started when the tile kernel was done, 62 us after they could; so 3 us after, and the step takes 194 us instead of 206.
struct RwGroupLds {
    static constexpr int NCH = RW_WIN / WAVE;
    uint32_t h_row[RW_HASH];
    int h_min[RW_HASH];
    uint16_t h_cnt[NCH * 64];
    uint64_t s_heads[NCH];
    uint16_t u_at[RW_WIN], u_rank[RW_WIN], s_start[RW_WIN + 4];
    int s_off[RW_OFF + 1], s_tmp[RW_NW], s_win[2];
    int bins[1];                                                   // [m1 + m3] rows per slice (or [spb] u of a slot)
};

template <bool CACHED>
__global__ __launch_bounds__(RW_T) void rw_group_kernel(Params p, int L, int win, const int64_t *__restrict__ offsets, int n_bags, RowsWs ws)
{
    constexpr int NCH = RwGroupLds::NCH, PER = RW_WIN / RW_T;
    extern __shared__ __align__(16) char rw_group_lds[];
    RwGroupLds &lds = *reinterpret_cast<RwGroupLds *>(rw_group_lds);
    uint32_t *h_row = lds.h_row;
    int *h_min = lds.h_min, *s_off = lds.s_off, *s_tmp = lds.s_tmp, *s_win = lds.s_win, *rw_bins = lds.bins;
    uint16_t *h_cnt = lds.h_cnt, *u_at = lds.u_at, *u_rank = lds.u_rank, *s_start = lds.s_start;
    uint64_t *s_heads = lds.s_heads;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, m13 = p.m1 + p.m3;
    if (!rw_find_window(p, win, ws, s_tmp, s_win)) return;          // uniform
    const int ostep = (n_bags + RW_OFF - 1) / RW_OFF;
    const bool search = offsets && !p.bagP;                        // (bags of one length are found without)
    if (search)
        for (int x = t; x <= RW_OFF; x += RW_T) s_off[x] = (int)offsets[min(x * ostep, n_bags)];
    for (int x = t; x < RW_HASH / 4; x += RW_T) {
        reinterpret_cast<uint4 *>(h_row)[x] = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
        reinterpret_cast<int4 *>(h_min)[x] = make_int4(0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff);
    }
    for (int x = t; x < NCH * 64; x += RW_T) h_cnt[x] = 0;
    __syncthreads();
    const int slice = s_win[0];
    const bool cached = CACHED && slice >= p.m2;                   // uniform
    if (cached) win = min(win, RW_CWIN);
    const int first = ws.goff[slice] + s_win[1] * win;
    const int n = min(win, ws.goff[slice + 1] - first), nch = (n + WAVE - 1) / WAVE;
    uint32_t myk[PER], myrow[PER];                                 // (LDS for three workgroups per compute unit)
    {
        uint32_t row[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = min(q * RW_T + t, n - 1);
            row[q] = ws.lrow[first + i];
            myk[q] = ws.lk[first + i];
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = q * RW_T + t;
            if (i >= n) continue;
            myrow[q] = row[q];
            uint32_t h = cache_hash(row[q], RW_HASH - 1);
            for (;;) {                                             // ends: at most RW_WIN rows in RW_HASH places
                uint32_t old = *(volatile uint32_t *)&h_row[h];    // (read first: a hot row's positions would queue up for one place)
                if (old == 0xffffffffu) old = atomicCAS(&h_row[h], 0xffffffffu, row[q]);
                if (old == 0xffffffffu || old == row[q]) break;
                h = (h + 1) & (RW_HASH - 1);
            }
            if (*(volatile int *)&h_min[h] > i) atomicMin(&h_min[h], i);
            u_at[i] = (uint16_t)h;
        }
    }
    __syncthreads();
    for (int ch = w; ch < nch; ch += RW_NW) {
        const int i = ch * WAVE + lane;
        const uint64_t head = __ballot(i < n && h_min[u_at[min(i, n - 1)]] == i);
        if (lane == 0) s_heads[ch] = head;
    }
    __syncthreads();
    int D = 0;
    for (int c = 0; c < nch; ++c) {
        const uint64_t head = s_heads[c];
        if ((c & (RW_NW - 1)) == w && ((head >> lane) & 1)) h_min[u_at[c * WAVE + lane]] = D + (int)__popcll(head & lanemask_lt());
        D += (int)__popcll(head);
    }
    __syncthreads();
    // numbers of the entries, entries of every number (at most RW_WIN numbers)
    uint32_t *count = h_row;                                       // then: its number among those with several entries
    constexpr uint32_t ONE = 0xffffu;
    for (int x = t; x < RW_WIN; x += RW_T) count[x] = 0u;
    __syncthreads();
    for (int i = t; i < n; i += RW_T) {
        const int num = h_min[u_at[i]];
        u_at[i] = (uint16_t)num;
        atomicAdd(&count[num], 1u);
    }
    __syncthreads();
    int M;
    {
        uint32_t c[PER];
        int sum = 0, several = 0, total;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            c[q] = count[t * PER + q];
            sum += (int)c[q];
            several += c[q] > 1u;
        }
        int at = rw_scan(sum, s_tmp, &total), m = rw_scan(several, s_tmp, &M);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int num = t * PER + q;
            if (num <= D) s_start[num] = (uint16_t)at;
            count[num] = c[q] > 1u ? (uint32_t)m : ONE;
            at += (int)c[q];
            m += c[q] > 1u;
        }
        if (t == 0) s_start[D] = (uint16_t)n;
    }
    // entries of a row with several: their places by a stable counting sort over 64 such rows at a time
    for (int m0 = 0; m0 < M; m0 += 64) {                           // uniform
        if (m0) {
            __syncthreads();
            for (int x = t; x < nch * 64; x += RW_T) h_cnt[x] = 0;
        }
        __syncthreads();
        for (int ch = w; ch < nch; ch += RW_NW) {
            const int i = ch * WAVE + lane, v = i < n ? (int)count[u_at[i]] - m0 : -1;
            const bool in = (unsigned)v < 64u;
            uint64_t same = __ballot(in);
            if (!same) continue;                                   // uniform
#pragma unroll
            for (int bit = 0; bit < 6; ++bit) {
                const uint64_t bal = __ballot((v >> bit) & 1);
                same &= (v >> bit) & 1 ? bal : ~bal;
            }
            if (in) {
                const int rank = (int)__popcll(same & lanemask_lt());
                u_rank[i] = (uint16_t)rank;
                if (rank == 0) h_cnt[ch * 64 + v] = (uint16_t)__popcll(same);
            }
        }
        __syncthreads();
        if (w == 0) {                                              // lane = row: counts of the chunks to places
            int sum = 0;
            for (int c = 0; c < nch; ++c) {
                const int x = h_cnt[c * 64 + lane];
                h_cnt[c * 64 + lane] = (uint16_t)sum;
                sum += x;
            }
        }
        __syncthreads();
        for (int i = t; i < n; i += RW_T) {
            const int v = (int)count[u_at[i]] - m0;
            if ((unsigned)v < 64u) u_rank[i] = (uint16_t)(h_cnt[(i >> 6) * 64 + v] + u_rank[i]);
        }
    }
    __syncthreads();
    const int room = cached ? ws.spb : m13;
    for (int x = t; x < room; x += RW_T) rw_bins[x] = cached ? -1 : 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = q * RW_T + t;
        if (i >= n) continue;
        const int k = (int)myk[q], num = u_at[i];
        int bag = k;
        if (offsets) {
            if (search) {
                int lo = 0, hi = RW_OFF;                           // last sample with offset <= k
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_off[mid] <= k) lo = mid; else hi = mid;
                }
                bag = min(lo * ostep, n_bags - 1);
                int b1 = min(bag + ostep, n_bags);
                while (b1 - bag > 1) {
                    const int mid = (bag + b1) >> 1;
                    if (offsets[mid] <= (int64_t)k) bag = mid; else b1 = mid;
                }
            } else {
                bag = grp_bag(p, offsets, n_bags, k);
            }
        }
        const int at = first + s_start[num] + (count[num] != ONE ? (int)u_rank[i] : 0);
        ws.gkb[at] = make_int2(k, bag);
        ws.gu[at] = first + num;
        const bool head = (s_heads[i >> 6] >> (i & 63)) & 1;
        if (cached) {
            if (head) {
                const int slot = ~ws.inv[k];
                ws.rec[first + num] = make_int4(slot, -1, first + s_start[num], s_start[num + 1] - s_start[num]);
                rw_bins[slot / RW_CBINS] = first + num;
            }
        } else {
            ws.inv[k] = first + num;
            if (head) {
                int i1, i2, i3;
                decode_f64(p, myrow[q], i1, i2, i3);
                ws.rec[first + num] = make_int4(i1, i3, first + s_start[num], s_start[num + 1] - s_start[num]);
                atomicAdd(&rw_bins[i1], 1);
                atomicAdd(&rw_bins[p.m1 + i3], 1);
            }
        }
        if (i >= D) ws.rec[first + i] = make_int4(0, 0, 0, 0);     // unused places
    }
    __syncthreads();
    for (int x = t; x < m13; x += RW_T) ws.hist2[(size_t)blockIdx.x * m13 + x] = cached ? 0u : (uint32_t)rw_bins[x];
    if (cached)
        for (int x = t; x < ws.spb; x += RW_T) ws.cu[(size_t)blockIdx.x * ws.spb + x] = rw_bins[x];
    if (t == 0) {
        ws.wd[blockIdx.x] = D;
        ws.wfirst[blockIdx.x] = first;
        ws.wslice[blockIdx.x] = slice;
    }
}

// Workgroups before the last: for SB bins each (slices of the first and third core) the windows' counts become the sums of the
// earlier windows, NG groups of threads sharing the windows.  The last one numbers the tiles.  Many windows (long streams, caches)
// take more groups: with 16 the 650 windows of a cached stream of 163,840 are six round trips one after the other, 8-9 us, with 64
// two, 6; few windows, as many workgroups as that needs only get in the way of what runs beside them (8,192 positions: step 91 / 93 us).
constexpr int RW_SBINS = 32, RW_SBINS_LONG = 8;
template <int SB>
__global__ __launch_bounds__(RW_T) void rw_scan_kernel(Params p, int tp, RowsWs ws)
{
    constexpr int NG = RW_T / SB;
    __shared__ uint32_t s_sum[NG][SB];
    __shared__ int s_tmp[RW_NW];
    const int t = threadIdx.x, m13 = p.m1 + p.m3, nw = *ws.nwin;
    if (blockIdx.x + 1 < gridDim.x) {
        constexpr int NF = 8;
        const int b = t % SB, g = t / SB, bin = (int)blockIdx.x * SB + b, per = (nw + NG - 1) / NG;
        const int w0 = min(nw, g * per), w1 = min(nw, w0 + per);
        const bool on = bin < m13;
        uint32_t *h = ws.hist2 + (on ? bin : 0);
        uint32_t sum = 0;
        for (int x = w0; x < w1; x += NF) {
            uint32_t v[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) v[q] = h[(size_t)min(x + q, w1 - 1) * m13];
#pragma unroll
            for (int q = 0; q < NF; ++q) sum += x + q < w1 ? v[q] : 0u;
        }
        s_sum[g][b] = sum;
        __syncthreads();
        uint32_t at = 0, all = 0;
#pragma unroll 16
        for (int q = 0; q < NG; ++q) {
            const uint32_t v = s_sum[q][b];
            if (q < g) at += v;
            all += v;
        }
        if (!on) return;
        if (g == 0) ws.tot2[bin] = all;
        for (int x = w0; x < w1; x += NF) {
            uint32_t v[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) v[q] = h[(size_t)min(x + q, w1 - 1) * m13];
#pragma unroll
            for (int q = 0; q < NF; ++q)
                if (x + q < w1) { h[(size_t)(x + q) * m13] = at; at += v[q]; }
        }
        return;
    }
    int base = 0;
    for (int w0 = 0; w0 < nw; w0 += RW_T) {                        // uniform
        const int x = w0 + t;
        const int s = x < nw ? ws.wslice[x] : 0, D = x < nw && s < p.m2 ? ws.wd[x] : 0, nt = (D + tp - 1) / tp;   // (no tiles of cached rows)
        int total;
        const int at = base + rw_scan(nt, s_tmp, &total);
        if (x < nw) {
            const int before = x ? ws.wslice[x - 1] : -1, first = ws.wfirst[x];
            for (int q = before + 1; q <= min(s, p.m2); ++q) ws.tile_base[q] = at;    // (slices without positions as well)
            for (int q = max(before + 1, p.m2); q <= s; ++q) ws.cwin[q - p.m2] = x;   // (bins of cached rows)
            for (int q = 0; q < nt; ++q) ws.tiles[at + q] = make_int4(s, first + q * tp, min(tp, D - q * tp), 0);
        }
        base += total;
    }
    const int last = nw ? ws.wslice[nw - 1] : -1;
    for (int q = last + 1 + t; q <= p.m2; q += RW_T) ws.tile_base[q] = base;
    if (ws.nb)
        for (int q = max(last + 1, p.m2) + t; q <= p.m2 + ws.nb; q += RW_T) ws.cwin[q - p.m2] = nw;
}

// The distinct rows of a window to their places among those of their slices of the first and of the third core.
template <bool CACHED>
__global__ __launch_bounds__(RW_T) void rw_lists_kernel(Params p, int bits1, int bits3, RowsWs ws)
{
    extern __shared__ __align__(16) uint32_t rw_lds[];             // [m13] starts, then [RW_NW][m13] 16-bit counts
    __shared__ int s_tmp[RW_NW];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, m13 = p.m1 + p.m3;
    if ((int)blockIdx.x >= *ws.nwin) return;                       // uniform
    uint32_t *start = rw_lds;
    uint16_t *cnt = reinterpret_cast<uint16_t *>(rw_lds + m13);
    const int D = ws.wd[blockIdx.x], first = ws.wfirst[blockIdx.x];
    constexpr int PB = RW_MAX_M13 / RW_T;                          // bins per thread: neighbouring ones
    {
        uint32_t v[PB];
        int sum = 0;
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            v[q] = t * PB + q < m13 ? ws.tot2[t * PB + q] : 0u;
            sum += (int)v[q];
        }
        int total;
        uint32_t at = (uint32_t)rw_scan(sum, s_tmp, &total);
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int bin = t * PB + q;
            if (bin < m13) {
                start[bin] = at + ws.hist2[(size_t)blockIdx.x * m13 + bin];
                if (blockIdx.x == 0) ws.off13[bin] = (int)at;
            }
            at += v[q];
        }
        if (blockIdx.x == 0 && t == 0) ws.off13[m13] = total;
    }
    if (CACHED && ws.wslice[blockIdx.x] >= p.m2) return;           // uniform: cached rows are in no list
    for (int x = t; x < RW_NW * m13; x += RW_T) cnt[x] = 0;
    __syncthreads();
    // wave w has the w-th eighth of the window's rows (whole chunks of 64)
    constexpr int NR = RW_WIN / RW_T;
    const int per = ((D + RW_NW - 1) / RW_NW + WAVE - 1) / WAVE * WAVE;
    int d1[NR], d3[NR], r1[NR], r3[NR], k0[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const int i = w * per + q * WAVE + lane;
        const bool in = q * WAVE < per && i < D;
        d1[q] = -1; d3[q] = 0; r1[q] = r3[q] = k0[q] = 0;
        if (in) {
            const int4 rc = ws.rec[first + i];
            d1[q] = rc.x; d3[q] = rc.y;
            k0[q] = ws.gkb[rc.z].x;
        }
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const bool in = d1[q] >= 0;
        const uint64_t any = __ballot(in);
        if (!any) continue;                                        // uniform
        auto rank = [&](int dg, int bits, int bin) {
            uint64_t same = any;
            for (int b = 0; b < bits; ++b) {                       // uniform
                const uint64_t bal = __ballot((dg >> b) & 1);
                same &= (dg >> b) & 1 ? bal : ~bal;
            }
            int r = 0;
            if (in) {
                const int old = cnt[w * m13 + bin], x = (int)__popcll(same & lanemask_lt());
                r = old + x;
                __builtin_amdgcn_wave_barrier();
                if (x == 0) cnt[w * m13 + bin] = (uint16_t)(old + (int)__popcll(same));
            }
            __builtin_amdgcn_wave_barrier();
            return r;
        };
        r1[q] = rank(d1[q], bits1, d1[q]);
        r3[q] = rank(d3[q], bits3, p.m1 + d3[q]);
    }
    __syncthreads();
    for (int bin = t; bin < m13; bin += RW_T) {
        int at = 0;
#pragma unroll
        for (int q = 0; q < RW_NW; ++q) {
            const int c = cnt[q * m13 + bin];
            cnt[q * m13 + bin] = (uint16_t)at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NR; ++q)
        if (d1[q] >= 0) {
            const int2 e = make_int2(first + w * per + q * WAVE + lane, k0[q]);
            ws.l13[start[d1[q]] + cnt[w * m13 + d1[q]] + r1[q]] = e;
            ws.l13[start[p.m1 + d3[q]] + cnt[w * m13 + p.m1 + d3[q]] + r3[q]] = e;
        }
}

static inline int rw_bits(int m)
{
    int b = 0;
    while ((1 << b) < m) ++b;
    return b;
}

// positions and rows grouped by second digit: two launches
static inline void rw_place(const Params &p, const int64_t *indices, int L, const CacheDev &cache, int tile, const RowsWs &ws, hipStream_t st)
{
    const int nblk = (L + tile - 1) / tile, bits = rw_bits(p.m2 + ws.nb);
    auto launch = [&](auto tl, auto cached) {
        constexpr int TILE = decltype(tl)::value;
        constexpr bool CACHED = decltype(cached)::value;
        hipLaunchKernelGGL((rw_count_kernel<TILE, CACHED>), dim3(nblk), dim3(TILE / RW_PER), 0, st, p, indices, L, cache, ws);
        hipLaunchKernelGGL((rw_scatter_kernel<TILE, CACHED>), dim3(nblk), dim3(TILE / RW_PER), 0, st, p, indices, L, nblk, bits, ws);
    };
    auto with_tile = [&](auto tl) {
        if (ws.nb) launch(tl, std::true_type{});
        else launch(tl, std::false_type{});
    };
    if (tile == RW_TILE_SHORT) with_tile(std::integral_constant<int, RW_TILE_SHORT>{});
    else with_tile(std::integral_constant<int, RW_TILE>{});
}

// Index-only part of a step: five launches.  tp: distinct rows per tile.
static inline hipError_t rw_prepare(const Params &p, const int64_t *indices, int L, const int64_t *offsets, int n_bags, const CacheDev &cache, int tp,
                                    const RowsWs &ws, hipStream_t st)
{
    const int nw = rw_windows(p, L, cache.K), m13 = p.m1 + p.m3;
    const size_t lds = (size_t)m13 * 4 + (size_t)RW_NW * m13 * 2;              // at most 80 KB
    static OncePerDevice once, once_cached, once_group, once_group_cached;
    const auto group = cache.K ? rw_group_kernel<true> : rw_group_kernel<false>;
    const auto lists = cache.K ? rw_lists_kernel<true> : rw_lists_kernel<false>;
    hipError_t e = allow_dynamic_lds(cache.K ? once_cached : once, (const void *)lists, RW_MAX_M13 * 4 + RW_NW * RW_MAX_M13 * 2);
    if (e != hipSuccess) return e;
    e = allow_dynamic_lds(cache.K ? once_group_cached : once_group, (const void *)group, sizeof(RwGroupLds) + RW_MAX_M13 * 4);
    if (e != hipSuccess) return e;
    rw_place(p, indices, L, cache, rw_tile(L), ws, st);
    // LDS: the counters of the digits, as many as there are (with 1,200 slices two workgroups share a compute unit, with 450
    // three; room for 4,096 of them, so that it is two for every table, makes no difference to the steps beside which they run:
    // 8,192 positions at rank 64 91.9 / 91.8 us, 60,000 at rank 32 134.1 / 134.2, of (2,2,4) 81.6 / 82.0, with a cache 80.8 / 81.1).
    const size_t bins = sizeof(RwGroupLds) + (size_t)(m13 > ws.spb ? m13 : ws.spb) * 4;
    hipLaunchKernelGGL(group, dim3(nw), dim3(RW_T), bins, st, p, L, rw_win(L), offsets, n_bags, ws);
    if (nw > 512) hipLaunchKernelGGL(rw_scan_kernel<RW_SBINS_LONG>, dim3((m13 + RW_SBINS_LONG - 1) / RW_SBINS_LONG + 1), dim3(RW_T), 0, st, p, tp, ws);
    else hipLaunchKernelGGL(rw_scan_kernel<RW_SBINS>, dim3((m13 + RW_SBINS - 1) / RW_SBINS + 1), dim3(RW_T), 0, st, p, tp, ws);
    hipLaunchKernelGGL(lists, dim3(nw), dim3(RW_T), lds, st, p, rw_bits(p.m1), rw_bits(p.m3), ws);
    return hipGetLastError();
}

}  // namespace tt
