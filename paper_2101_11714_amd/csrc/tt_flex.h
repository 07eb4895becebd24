// Forward and backward for the shapes without a compile-time configuration (any column factors and ranks within the
// limits of flex_supported): every size is a run-time value, the products of Eq. 4 run on the matrix cores all the same.
//
// Forward: a wave per bag, lane l owns V columns of the unfolded second core, T0 in registers, then through LDS to the
// second product (flex_fwd_kernel), where that is ahead of the plain kernel (flex_fwd_pays).
//
// Backward, two launches:
//   1. flex_g2_kernel: one workgroup per slice of the second core (times S for long streams, each on a part of the
//      positions).  It scans the indices for its positions, groups them by row, adds the upstream gradients of equal
//      rows up, and works on tiles of up to 64 stacked rows (row, j1) of distinct rows:
//          dT0' = dY C^T,   dG2 += A^T dT0',   P = dT0' Bm^T (the G1 gradient),   T0 = A Bm,   Q = T0^T dY (the G3 gradient),
//      the three large ones as fp32 MFMA 16x16x4 products with operands in LDS, up to 64 columns (whole values of j2)
//      at a time.  The slice gradient is finished on the spot; P and Q of a distinct row go to the workspace, filed under
//      the first position k of the row, and rec[k] says which slices they belong to.
//   2. flex_sum_kernel: one workgroup per slice of the first and of the third core scans rec for its rows and adds them
//      up in the order of k; more workgroups add the parts of the second core where S > 1.
// P and Q of every position of a long stream may need more room than there is: then the two launches are made several
// times, for as many positions as fit, and the sums so far wait in the workspace.  Results are the same bit for bit: lists
// are worked off wherever a pass may end, whether one does or not.  That costs a stream beyond FX_PIECE_BYTES something:
// 100,000 positions, (2,4,4) at rank 24 339 -> 357 us, (2,4,8) at rank 64 1,384 -> 1,598 us; in passes within 32 MiB the
// same calls take 460 and 6,250 us, with the plain kernels 10,500 and 64,400.
// No atomics; every sum has a fixed order, so results repeat bit for bit.
//
// What bounds it (4,096 positions, (4,4,4) at rank 16): latency.  A workgroup is a chain of index scan, list, gathers of
// gradients and slices (each a miss of the L2, which is cold at a kernel's start) and a few barriers, 14 us for the usual
// slice, 20 us for one of more than TP distinct rows or with a hot row; 200 workgroups leave each a compute unit of its
// own, hence 512 threads.  Whole step (forward 8, this 21, the sums 6 us): 885 us with the kernels of tt_generic.h, which
// contract row after row with barriers between any two steps, 39 us with these; (2,4,4) at rank 24 with 1-3 positions per
// bag 831 -> 47 us.
#pragma once

#include <type_traits>

#include "tt_common.h"
#include "tt_fast_bwd.h"

namespace tt {

constexpr int FX_T = 512, FX_NW = FX_T / WAVE;   // threads / waves of flex_g2_kernel
constexpr int FX_ROWS = 64;                      // stacked rows (distinct row, j1) of a tile
constexpr int FX_ROUND = 2048;                   // positions scanned per round
constexpr int FX_HASH = 4096;                    // places of the hash table that merges equal rows
constexpr int FX_CAP = FX_ROUND + 1024;          // list entries held before they are worked on
constexpr int FX_OFF = 2048;                     // samples of the offsets array kept in LDS
constexpr int FX_CW = 64, FX_LD = FX_CW + 4;     // columns of a pass; row stride in LDS (4 * odd: no bank conflicts on either operand)
constexpr int FX_LONG = 16;                      // a run of more equal rows is added up in pieces of that many
constexpr int FX_TILE = 3840;                    // values of the third core's slices, and of upstream gradients, of a tile
constexpr int FX_MAX_LDS = 114 * 1024;           // dynamic LDS of a tile at the limits of flex_supported (45 KB of static lists beside it)

struct FlexDims {
    int TP;              // distinct rows per tile
    int JB;              // values of j2 per pass
    int R1p, LDA;        // R1 rounded up to 16; row stride of the stacked G1 rows
    uint32_t mgSC;       // ceil(2^32 / sC)
    int S, seg;          // workgroups per slice of the second core (segments of the stream), positions of each
    int piece;           // a pass has this many positions or a multiple (of a segment: or what is left of it): whole
                         // segments, or a part of one.  Streams of up to `whole` positions take one pass.
    int whole;
    int lds_floats;      // of the tile area
};

static inline uint32_t magic_div(uint32_t d) { return d > 1 ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u; }

// Shapes these kernels take.  The limits keep a tile's operands in LDS (at most 114 KB, 45 KB of lists beside it).
static inline bool flex_supported(const Params &p)
{
    return p.R1 <= 64 && p.R2 <= 64 && p.n1 <= 16 && p.n2 * p.n3 <= 64 && p.N <= 256 && p.sC <= 1024 && p.n1 * p.cols <= 4096;
}

// P, Q and rec of a piece, where the static scratch memory has room for that; of the passes that a queried workspace allows.
// (The second: (4,4,4) at rank 16 starts a second pass beyond 516,000 positions.)
constexpr int FX_SEGMENTS = 16;                  // segments of a stream, at most
constexpr size_t FX_PIECE_BYTES = (size_t)16 << 20, FX_PASS_BYTES = (size_t)256 << 20;

static inline size_t flex_row_bytes(const Params &p) { return 8 + 4 * ((size_t)p.sA + p.sC); }

// piece_bytes: see FX_PIECE_BYTES; most: the largest number of segments
static inline FlexDims flex_dims(const Params &p, int64_t L, size_t piece_bytes, int most)
{
    FlexDims d;
    const int64_t rounds = (int64_t)(piece_bytes / flex_row_bytes(p) / FX_ROUND);
    d.whole = FX_ROUND * (int)(rounds < 1 ? 1 : rounds);
    d.TP = FX_ROWS / p.n1;
    if (d.TP > FX_TILE / p.sC) d.TP = FX_TILE / p.sC;
    if (d.TP > FX_TILE / p.N) d.TP = FX_TILE / p.N;
    d.JB = FX_CW / p.R2 > 1 ? FX_CW / p.R2 : 1;
    d.R1p = (p.R1 + 15) & ~15;
    d.LDA = d.R1p + 4;
    d.mgSC = magic_div((uint32_t)p.sC);
    // a workgroup of its own for every 8,192 positions of a slice (four scan rounds), at most 16
    int64_t s = (L + 8191) / 8192;
    s = s < 1 ? 1 : (s > most ? most : s);
    d.seg = (int)(((L + s - 1) / s + FX_ROUND - 1) / FX_ROUND * FX_ROUND);
    if (d.seg < FX_ROUND) d.seg = FX_ROUND;
    d.S = (int)(L > 0 ? (L + d.seg - 1) / d.seg : 1);
    d.piece = d.whole >= d.seg ? d.whole / d.seg * d.seg : d.whole;
    const int tile = FX_ROWS * (d.LDA + 2 * FX_LD) + d.R1p * FX_LD + 2 * ((d.TP * p.sC + 3) & ~3) + d.TP * p.N + 16;
    const int lists = 5 * FX_CAP + 2 * FX_HASH + FX_OFF + 8;   // the unsorted list and its hash table lie in the tile area
    d.lds_floats = tile > lists ? tile : lists;
    return d;
}

struct FlexWs {
    // (n: positions of a pass, at most)
    int2 *rec;           // [n] {i1, i3} of a position that stands for a distinct row, else {-1, -1}
    float *pbuf, *cbuf;  // [n][sA], [n][sC]: gradients of the first and third core's slices of that row
    float *part;         // [segments of a pass][m2][sB]
    float *acc;          // [m1][sA], [m3][sC], [m2][sB] (S > 1): sums of the passes so far
    size_t bytes;
};

// n: positions of a pass; several: a call of more than one
static inline FlexWs flex_ws_layout(void *ws, const Params &p, const FlexDims &d, int64_t n, int parts, bool several)
{
    FlexWs w;
    char *base = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *q = base ? base + off : nullptr; off += (bytes + 255) & ~(size_t)255; return q; };
    if (n < 1) n = 1;
    w.rec = (int2 *)take((size_t)n * 8);
    w.pbuf = (float *)take((size_t)n * p.sA * 4);
    w.cbuf = (float *)take((size_t)n * p.sC * 4);
    w.part = (float *)take((size_t)parts * p.m2 * p.sB * 4);
    w.acc = (float *)take(!several ? 0 : ((size_t)p.m1 * p.sA + (size_t)p.m3 * p.sC + (d.S > 1 ? (size_t)p.m2 * p.sB : 0)) * 4);
    w.bytes = off;
    return w;
}

// for passes of `pass` positions of a stream of L
static inline FlexWs flex_ws_layout(void *ws, const Params &p, const FlexDims &d, int64_t L, int64_t pass)
{
    const int64_t n = L < pass ? L : pass;
    return flex_ws_layout(ws, p, d, n, n < 1 ? 1 : (int)((n + d.seg - 1) / d.seg), pass < L);
}

// the least that a call can do with
static inline size_t flex_ws_least(const Params &p, const FlexDims &d, int64_t L)
{
    return flex_ws_layout(nullptr, p, d, L, L <= d.whole ? L : d.piece).bytes;
}

// what a query answers: enough for passes of FX_PASS_BYTES (or a piece), for every length up to L
static inline size_t flex_ws_query(const Params &p, const FlexDims &d, int64_t L)
{
    int64_t n = (int64_t)(FX_PASS_BYTES / flex_row_bytes(p));
    if (n < d.whole) n = d.whole;
    const int64_t parts = (L + 8191) / 8192;                     // (d.S may fall where the segments get longer)
    return flex_ws_layout(nullptr, p, d, L < n ? L : n, parts < 1 ? 1 : (parts < FX_SEGMENTS ? (int)parts : FX_SEGMENTS), true).bytes;
}

// Positions of a pass for `room` bytes: all, or as many pieces as fit (whole segments where a piece is shorter); 0: too
// little room.
static inline int64_t flex_pass(const Params &p, const FlexDims &d, int64_t L, size_t room)
{
    auto fits = [&](int64_t n) { return flex_ws_layout(nullptr, p, d, L, n).bytes <= room; };
    if (fits(L)) return L;
    if (L <= d.whole) return 0;
    if (d.piece >= d.seg || fits(d.seg)) {
        const int64_t unit = d.piece >= d.seg ? d.piece : d.seg;
        int64_t n = L / unit * unit;                              // (at most FX_SEGMENTS of them)
        while (n > 0 && !fits(n)) n -= unit;
        return n;
    }
    int64_t lo = 0, hi = d.seg / d.piece + 1;                     // pieces: lo fit (or none), hi do not
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (mid * d.piece < d.seg && fits(mid * d.piece)) lo = mid; else hi = mid;
    }
    return lo * d.piece;
}

struct FlexArgs {
    Params p;
    FlexDims d;
    const float *G1, *G2, *G3;
    const int64_t *indices, *offsets;
    int L, n_bags;
    const float *alpha;
    const int32_t *slot;
    const float *go;
    const float *src[3];     // dst[k] = src[k] + mul * gradient
    float *dst[3];
    float mul;
    FlexWs w;
    // the pass: positions [k0, k1) (whole segments, or a part of one), whether it continues a segment, whether it is the
    // first and the last one, and whether the parts of the second core are added up after it (never, where S = 1)
    int k0, k1;
    bool cont, first, fin, fold;
};

// V4: n3 = 4 and both ranks are multiples of 4, so that everything moves as float4.  ONE: a stream of up to `whole` positions,
// which takes one pass (without what several need the two kernels of a step of 4,096 positions take 28 us instead of 29: it is cold
// kernel arguments and instructions).
template <bool V4, bool ONE>
__global__ __launch_bounds__(FX_T) void flex_g2_kernel(FlexArgs a)
{
    extern __shared__ __align__(16) float fx_lds[];
    __shared__ int s_k[FX_CAP], s_bag[FX_CAP];                              // sorted list: position, bag
    __shared__ uint16_t s_start[FX_CAP + 2];                                // first entries of its runs
    __shared__ uint32_t s_row[FX_CAP];                                      // rows of the runs
    __shared__ int s_cnt[2][FX_NW];
    __shared__ uint64_t s_heads[FX_CAP / WAVE];
    __shared__ int s_re[FX_ROWS], s_rj[FX_ROWS], s_piece[FX_ROWS + 1];                            // stacked row -> distinct row of the tile, j1
    const Params &p = a.p;
    const FlexDims &d = a.d;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = t & 15, q16 = (t >> 4) & 3, gid = t >> 4;
    const int n1 = p.n1, n2 = p.n2, n3 = V4 ? 4 : p.n3, R1 = p.R1, R2 = p.R2, N = p.N, cols = p.cols, sA = p.sA, sC = p.sC, LDA = d.LDA;
    const int k0 = ONE ? 0 : a.k0, k1 = ONE ? a.L : a.k1;
    const bool fin = ONE || a.fin;
    const int i2 = blockIdx.x % p.m2, sp = blockIdx.x / p.m2;
    const int k_lo = k0 + sp * d.seg, k_hi = min(k1, k_lo + d.seg);

    float *As = fx_lds;                              // [64][LDA]    stacked rows of G1
    float *dT = As + FX_ROWS * LDA;                  // [64][FX_LD]  dT0'
    float *Ts = dT + FX_ROWS * FX_LD;                // [64][FX_LD]  T0
    float *Bs = Ts + FX_ROWS * FX_LD;                // [R1p][FX_LD] Bm
    float *Cs = Bs + d.R1p * FX_LD;                  // [TP][sC]     slices of G3
    float *Qs = Cs + ((d.TP * sC + 3) & ~3);         // [TP][sC]     their gradients
    float *Ys = Qs + ((d.TP * sC + 3) & ~3);         // [TP][N]      summed upstream gradients
    int *u_k = reinterpret_cast<int *>(fx_lds);      // the list before it is sorted
    uint32_t *u_r = reinterpret_cast<uint32_t *>(u_k) + FX_CAP;
    int *u_at = reinterpret_cast<int *>(u_r) + FX_CAP, *u_rank = u_at + FX_CAP;
    uint32_t *h_row = reinterpret_cast<uint32_t *>(u_rank) + FX_CAP;   // [FX_HASH] and the hash table ...
    int *h_min = reinterpret_cast<int *>(h_row) + FX_HASH;
    int *h_cnt = h_min + FX_HASH;                    // [FX_CAP / 64][64] ... and the counts of the sort
    int *s_off = h_cnt + FX_CAP;                     // [FX_OFF + 1] every ostep-th offset, for the bags of the positions

    const int ostep = (a.n_bags + FX_OFF - 1) / FX_OFF;
    const bool search = a.offsets && !p.bagP;        // (bags of one length are found without)
    auto load_offsets = [&]() {
        for (int x = t; x <= FX_OFF; x += FX_T) s_off[x] = (int)a.offsets[min(x * ostep, a.n_bags)];
    };
    if (t < FX_ROWS) {
        const int e = t / n1;
        s_re[t] = e < d.TP ? e : -1;
        s_rj[t] = t - e * n1;
    }
    // rows of the passes below that this thread works on, and its columns of a pass
    int cj[FX_CW / 16], cb[FX_CW / 16];
#pragma unroll
    for (int i = 0; i < FX_CW / 16; ++i) {
        cj[i] = (l16 + 16 * i) / R2;
        cb[i] = (l16 + 16 * i) - cj[i] * R2;
    }

    bool in_part = !ONE && a.cont;                   // this workgroup's slice gradient so far is in `part`
    const float *src2 = a.src[1] + (size_t)i2 * p.sB;
    float *dst2 = a.dst[1] + (size_t)i2 * p.sB;
    float *part = a.w.part + ((size_t)sp * p.m2 + i2) * p.sB;
    const float *G2s = a.G2 + (size_t)i2 * p.sB;

    // Bm for one pass, in registers: rows gid and gid + 32, four columns (rows past R1: zeros; columns past the pass: any)
    float rbm[2][4];
    auto fetch_bm = [&](int jc) {
        const int cw = min(d.JB, n2 - jc) * R2;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = gid + FX_T / 16 * i;
            const float *B = G2s + (size_t)min(r, R1 - 1) * cols + jc * R2;
            if constexpr (V4) {
                const float4 v = *reinterpret_cast<const float4 *>(B + min(4 * l16, cw - 4));
                rbm[i][0] = v.x; rbm[i][1] = v.y; rbm[i][2] = v.z; rbm[i][3] = v.w;
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x) rbm[i][x] = B[min(4 * l16 + x, cw - 1)];
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) rbm[i][x] = r < R1 ? rbm[i][x] : 0.f;
        }
    };

    auto bag_find = [&](int k) {
        if (!a.offsets) return k;
        if (p.bagP) {
            int g = (int)fast_div((uint32_t)k, p.bagP, p.mgP);
            g = g < a.n_bags ? g : a.n_bags - 1;
            if (a.offsets[g] <= (int64_t)k && (int64_t)k < a.offsets[g + 1]) return g;
            return bag_of(a.offsets, a.n_bags, k);
        }
        int lo = 0, hi = FX_OFF;                     // last sample with offset <= k
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_off[mid] <= k) lo = mid; else hi = mid;
        }
        int b0 = min(lo * ostep, a.n_bags - 1), b1 = min(b0 + ostep, a.n_bags);
        while (b1 - b0 > 1) {
            const int mid = (b0 + b1) >> 1;
            if (a.offsets[mid] <= (int64_t)k) b0 = mid; else b1 = mid;
        }
        return b0;
    };

    // the distinct rows [d0, d0 + nt) of the sorted list
    auto tile = [&](int d0, int nt, bool last) {
        const int nrow = nt * n1, nrb = (nrow + 15) >> 4;
        // The operands are loaded into registers first, all loads in flight together with those of the upstream gradients.
        // Stacked rows of G1 (rows past the end and columns past R1: zeros): four columns per lane, two rows ...
        float ra[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = gid + FX_T / 16 * i;
            const bool on = r < nrow;
            int x1 = 0, x2, x3;
            if (on) decode_f64(p, s_row[d0 + s_re[r]], x1, x2, x3);
            const float *A = a.G1 + (size_t)x1 * sA + (on ? s_rj[r] * R1 : 0);
            if constexpr (V4) {
                const float4 v = *reinterpret_cast<const float4 *>(A + min(4 * l16, R1 - 4));
                ra[i][0] = v.x; ra[i][1] = v.y; ra[i][2] = v.z; ra[i][3] = v.w;
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x) ra[i][x] = A[min(4 * l16 + x, R1 - 1)];
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) ra[i][x] = on && 4 * l16 + x < R1 ? ra[i][x] : 0.f;
        }
        // ... and slices of G3 (at most FX_TILE values): two float4 per thread
        float rc[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int x = min(4 * (t + FX_T * i), nt * sC - 1);
            if constexpr (V4) {
                const int xx = x & ~3, e = (int)fast_div((uint32_t)xx, (uint32_t)sC, d.mgSC);
                int x1, x2, x3;
                decode_f64(p, s_row[d0 + e], x1, x2, x3);
                const float4 v = *reinterpret_cast<const float4 *>(a.G3 + (size_t)x3 * sC + (xx - e * sC));
                rc[i][0] = v.x; rc[i][1] = v.y; rc[i][2] = v.z; rc[i][3] = v.w;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int xx = min(x + q, nt * sC - 1), e = (int)fast_div((uint32_t)xx, (uint32_t)sC, d.mgSC);
                    int x1, x2, x3;
                    decode_f64(p, s_row[d0 + e], x1, x2, x3);
                    rc[i][q] = a.G3[(size_t)x3 * sC + (xx - e * sC)];
                }
            }
        }
        // the summed upstream gradient of every distinct row, entries in list order; VW values per lane
        auto sum_dy = [&](auto vw) {
            constexpr int VW = decltype(vw)::value;
            const int nv = N / VW;
            int lp = 1, sh = 0;                                   // lanes per row: a power of two
            while (lp < nv) { lp <<= 1; ++sh; }
            const int f = t & (lp - 1), g = t >> sh, ng = FX_T >> sh;
            const bool on = f < nv;
            const float *gof = a.go + (on ? VW * f : 0);
            auto add = [&](auto nb, float (&s)[VW], int first, int end, int step) {
                constexpr int NB = decltype(nb)::value;           // loads in flight
                for (int i = first; i < end; i += NB * step) {
                    float x[NB][VW], wt[NB];
#pragma unroll
                    for (int q = 0; q < NB; ++q) {
                        const int ii = min(i + q * step, end - 1);
                        wt[q] = i + q * step < end ? (a.alpha ? a.alpha[s_k[ii]] : 1.f) : 0.f;
                        load_vec<VW>(gof + (size_t)s_bag[ii] * N, x[q]);
                    }
#pragma unroll
                    for (int q = 0; q < NB; ++q)
                        if (i + q * step < end) {
#pragma unroll
                            for (int v = 0; v < VW; ++v) s[v] = fmaf(wt[q], x[q][v], s[v]);
                        }
                }
            };
            for (int e = g; e < nt; e += ng) {
                const int b = s_start[d0 + e], c = s_start[d0 + e + 1];
                if (c - b > FX_LONG) continue;
                float s[VW] = {};
                if (c - b <= 2) add(std::integral_constant<int, 2>{}, s, b, c, 1);
                else add(std::integral_constant<int, 8>{}, s, b, c, 1);
                if (on) store_vec<VW>(Ys + e * N + VW * f, s);
            }
            // Longer runs in pieces of FX_LONG entries, all pieces of all runs side by side, then piece after piece.  The
            // partial sums lie in the dT / Ts area; what does not fit there (wide rows, thousands of entries) goes in turns.
            const int room = 2 * FX_ROWS * FX_LD / N;
            if (w == 0) {
                const int len = lane < nt ? s_start[d0 + lane + 1] - s_start[d0 + lane] : 0;
                int inc = len > FX_LONG ? (len + FX_LONG - 1) / FX_LONG : 0;
                const int own = inc;
#pragma unroll
                for (int q = 1; q < 64; q <<= 1) {
                    const int o = __shfl_up(inc, q);
                    if (lane >= q) inc += o;
                }
                if (lane <= nt) s_piece[lane] = inc - own;        // (lane nt has no pieces of its own)
                if (nt == WAVE && lane == WAVE - 1) s_piece[nt] = inc;
            }
            __syncthreads();
            const int np = s_piece[nt];
            for (int p0 = 0; p0 < np; p0 += room) {               // uniform
                const int p1 = min(np, p0 + room);
                for (int pc = p0 + g; pc < p1; pc += ng) {
                    int lo = 0, hi = nt;                          // last e with s_piece[e] <= pc (runs without pieces share their start)
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (s_piece[mid] <= pc) lo = mid; else hi = mid;
                    }
                    const int b = s_start[d0 + lo] + (pc - s_piece[lo]) * FX_LONG, c = min(b + FX_LONG, (int)s_start[d0 + lo + 1]);
                    float s[VW] = {};
                    add(std::integral_constant<int, 8>{}, s, b, c, 1);
                    if (on) store_vec<VW>(dT + (pc - p0) * N + VW * f, s);
                }
                __syncthreads();
                for (int e = g; e < nt; e += ng) {
                    const int b = max(s_piece[e], p0), c = min(s_piece[e + 1], p1);
                    if (b >= c || !on) continue;
                    float tot[VW] = {};
                    if (b > s_piece[e]) load_vec<VW>(Ys + e * N + VW * f, tot);
                    for (int q = b; q < c; ++q) {
                        float x[VW];
                        load_vec<VW>(dT + (q - p0) * N + VW * f, x);
#pragma unroll
                        for (int v = 0; v < VW; ++v) tot[v] += x[v];
                    }
                    store_vec<VW>(Ys + e * N + VW * f, tot);
                }
                __syncthreads();
            }
        };
        sum_dy(std::integral_constant<int, V4 ? 4 : 1>{});

#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = gid + FX_T / 16 * i, x = 4 * (t + FX_T * i);
            if (r < 16 * nrb && 4 * l16 < d.R1p) *reinterpret_cast<float4 *>(As + r * LDA + 4 * l16) = make_float4(ra[i][0], ra[i][1], ra[i][2], ra[i][3]);
            if (x < d.TP * sC) *reinterpret_cast<float4 *>(Cs + x) = make_float4(rc[i][0], rc[i][1], rc[i][2], rc[i][3]);
        }

        // P: row block w & 3, column blocks (w >> 2) + 2 i
        mfma4_t accp[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        const int prb = w & 3;
        for (int jc = 0; jc < n2; jc += d.JB) {
            const int jn = min(d.JB, n2 - jc), cw = jn * R2, nb2 = (cw + 15) >> 4;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = gid + FX_T / 16 * i;
                if (r < d.R1p && 4 * l16 < 16 * nb2)
                    *reinterpret_cast<float4 *>(Bs + r * FX_LD + 4 * l16) =
                        make_float4(4 * l16 + 0 < cw ? rbm[i][0] : 0.f, 4 * l16 + 1 < cw ? rbm[i][1] : 0.f,
                                    4 * l16 + 2 < cw ? rbm[i][2] : 0.f, 4 * l16 + 3 < cw ? rbm[i][3] : 0.f);
            }
            __syncthreads();                                      // Ys, Cs, As are in place (first pass)
            fetch_bm(jc + d.JB < n2 ? jc + d.JB : 0);             // the next pass, or the next tile's first one
            for (int r = gid; r < 16 * nrb; r += FX_T / 16) {
                const bool on = r < nrow;
                const int e = on ? s_re[r] : 0, j1 = on ? s_rj[r] : 0;
                const float *y = Ys + e * N + (j1 * n2 + jc) * n3, *cc = Cs + e * sC;
#pragma unroll
                for (int i = 0; i < FX_CW / 16; ++i)
                    if (i < nb2) {                                // uniform
                        const bool in = on && l16 + 16 * i < cw;
                        const float *yy = y + (in ? cj[i] : 0) * n3, *c3 = cc + (in ? cb[i] : 0) * n3;
                        float s = 0.f;
                        if constexpr (V4) {
                            const float4 y4 = *reinterpret_cast<const float4 *>(yy), c4 = *reinterpret_cast<const float4 *>(c3);
                            s = fmaf(y4.x, c4.x, fmaf(y4.y, c4.y, fmaf(y4.z, c4.z, y4.w * c4.w)));
                        } else {
                            for (int j = 0; j < n3; ++j) s = fmaf(yy[j], c3[j], s);
                        }
                        dT[r * FX_LD + l16 + 16 * i] = in ? s : 0.f;
                    }
            }
            // T0 = A Bm (needs Bs and As only)
            for (int id = w; id < nrb * nb2; id += FX_NW) {
                const int rb = id % nrb, bb = id / nrb;
                mfma4_t acc = {0.f, 0.f, 0.f, 0.f};
                const float *ar = As + (16 * rb + l16) * LDA + 4 * q16, *br = Bs + 4 * q16 * FX_LD + 16 * bb + l16;
                for (int s = 0; s < d.R1p; s += 16) {
                    const float4 av = *reinterpret_cast<const float4 *>(ar + s);
                    const float *b4 = br + s * FX_LD;
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, b4[0], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, b4[FX_LD], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, b4[2 * FX_LD], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, b4[3 * FX_LD], acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) Ts[(16 * rb + 4 * q16 + r) * FX_LD + 16 * bb + l16] = acc[r];
            }
            __syncthreads();
            // dG2 = A^T dT0'
            const int nra = d.R1p >> 4;
            for (int id = w ^ (FX_NW / 2); id < nra * nb2; id += FX_NW) {   // (the waves without rows of P below first)
                const int ab = id % nra, bb = id / nra;
                mfma4_t acc = {0.f, 0.f, 0.f, 0.f};
                const bool final = last && d.S == 1;
                int off[4];
                bool in[4];
                float old[4], sofar[4];                          // (fetched before the products)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int aa = 16 * ab + 4 * q16 + r, c = 16 * bb + l16;
                    in[r] = aa < R1 && c < cw;
                    off[r] = in[r] ? aa * cols + jc * R2 + c : 0;
                    old[r] = final ? src2[off[r]] : 0.f;
                    sofar[r] = in_part ? part[off[r]] : 0.f;
                }
                const float *ar = As + q16 * LDA + 16 * ab + l16, *br = dT + q16 * FX_LD + 16 * bb + l16;
                for (int s = 0; s < 16 * nrb; s += 16) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[(s + 4 * u) * LDA], br[(s + 4 * u) * FX_LD], acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (in[r]) {
                        const float s = sofar[r] + acc[r];
                        if (final) dst2[off[r]] = fmaf(a.mul, s, old[r]);
                        else part[off[r]] = s;
                    }
            }
            // P += dT0' Bm^T
            if (prb < nrb) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int ab = (w >> 2) + 2 * i;
                    if (ab < nra) {
                        const float *ar = dT + (16 * prb + l16) * FX_LD + 4 * q16, *br = Bs + (16 * ab + l16) * FX_LD + 4 * q16;
                        for (int s = 0; s < 16 * nb2; s += 16) {
                            const float4 av = *reinterpret_cast<const float4 *>(ar + s), bv = *reinterpret_cast<const float4 *>(br + s);
                            accp[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, accp[i], 0, 0, 0);
                            accp[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, accp[i], 0, 0, 0);
                            accp[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, bv.z, accp[i], 0, 0, 0);
                            accp[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, bv.w, accp[i], 0, 0, 0);
                        }
                    }
                }
            }
            // Q[e][b][j3] (+)= sum_(j1, j2 of the pass) T0[(e,j1)][(j2,b)] dY[e][(j1,j2)][j3]
            const int nbb = (R2 + 15) >> 4;
            for (int id = gid; id < nt * nbb; id += FX_T / 16) {
                const int e = id / nbb, b = 16 * (id - e * nbb) + l16;
                if (b >= R2) continue;
                for (int j3 = 0; j3 < n3; j3 += 4) {
                    float s[4] = {0.f, 0.f, 0.f, 0.f};
                    for (int j1 = 0; j1 < n1; ++j1)
                        for (int jj = 0; jj < jn; ++jj) {
                            const float tv = Ts[(e * n1 + j1) * FX_LD + jj * R2 + b];
                            const float *y = Ys + e * N + (j1 * n2 + jc + jj) * n3 + j3;
                            if constexpr (V4) {
                                const float4 y4 = *reinterpret_cast<const float4 *>(y);
                                s[0] = fmaf(tv, y4.x, s[0]); s[1] = fmaf(tv, y4.y, s[1]);
                                s[2] = fmaf(tv, y4.z, s[2]); s[3] = fmaf(tv, y4.w, s[3]);
                            } else {
#pragma unroll
                                for (int x = 0; x < 4; ++x) s[x] = fmaf(tv, y[j3 + x < n3 ? x : 0], s[x]);
                            }
                        }
                    // the sums over the passes stay in LDS, the last pass sends them out
                    float *q = Qs + e * sC + b * n3 + j3;
                    if (jc > 0) {
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            if (j3 + x < n3) s[x] += q[x];
                    }
                    auto put = [&](float *o) __attribute__((always_inline)) {
                        if constexpr (V4) {
                            *reinterpret_cast<float4 *>(o) = make_float4(s[0], s[1], s[2], s[3]);
                        } else {
#pragma unroll
                            for (int x = 0; x < 4; ++x)
                                if (j3 + x < n3) o[x] = s[x];
                        }
                    };
                    if (jc + jn < n2) put(q);
                    else put(a.w.cbuf + (size_t)(s_k[s_start[d0 + e]] - k0) * sC + b * n3 + j3);
                }
            }
            __syncthreads();                                      // the tile area is rewritten
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int aa = 16 * ((w >> 2) + 2 * i) + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * prb + 4 * q16 + r;
                if (row < nrow && aa < R1) a.w.pbuf[(size_t)(s_k[s_start[d0 + s_re[row]]] - k0) * sA + s_rj[row] * R1 + aa] = accp[i][r];
            }
        }
    };

    // Groups the n entries of the list by row, rows in the order of their first entries and entries in list order, and
    // works through the distinct rows.  Rows meet in a hash table in LDS, where the smallest list index of a row makes
    // that entry the row's head; the heads are numbered in list order and the entries placed by a stable counting sort
    // over 64 of those numbers at a time.  (A rank sort by comparing every pair took 16 us for the 477 entries of a hot
    // slice, this 2 us.)
    auto work = [&](int n, bool last) {
        if (search && in_part) load_offsets();                    // (a tile has been worked on since they were loaded)
        const int nch = (n + WAVE - 1) / WAVE;                    // chunks of 64 entries: wave w has chunks w, w + 8, ...
        for (int x = t; x < nch * 64; x += FX_T) h_cnt[x] = 0;
        for (int x = t; x < FX_HASH / 4; x += FX_T) {
            reinterpret_cast<uint4 *>(h_row)[x] = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
            reinterpret_cast<int4 *>(h_min)[x] = make_int4(0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff);
        }
        __syncthreads();
        // (rolled loops, what a thread keeps of an entry is in LDS: this kernel's length is instruction fetches that every
        // compute unit pays for)
#pragma unroll 1
        for (int i = t; i < n; i += FX_T) {
            const uint32_t my = u_r[i];
            uint32_t h = cache_hash(my, FX_HASH - 1);
            for (;;) {                                            // ends: at most FX_CAP rows in FX_HASH places
                const uint32_t old = atomicCAS(&h_row[h], 0xffffffffu, my);
                if (old == 0xffffffffu || old == my) break;
                h = (h + 1) & (FX_HASH - 1);
            }
            atomicMin(&h_min[h], i);
            u_at[i] = (int)h;                                     // place in the table, later the number of the row
        }
        __syncthreads();
#pragma unroll 1
        for (int ch = w; ch < nch; ch += FX_NW) {
            const int i = ch * WAVE + lane;
            const uint64_t head = __ballot(i < n && h_min[u_at[min(i, n - 1)]] == i);
            if (lane == 0) s_heads[ch] = head;
        }
        __syncthreads();
        int D = 0;
#pragma unroll 1
        for (int c = 0; c < nch; ++c) {
            const uint64_t head = s_heads[c];
            if ((c & (FX_NW - 1)) == w && ((head >> lane) & 1)) h_min[u_at[c * WAVE + lane]] = D + (int)__popcll(head & lanemask_lt());
            D += (int)__popcll(head);
        }
        __syncthreads();
#pragma unroll 1
        for (int i = t; i < n; i += FX_T) u_at[i] = h_min[u_at[i]];
        int placed = 0;
#pragma unroll 1
        for (int d0 = 0; d0 < D; d0 += 64) {                      // uniform
#pragma unroll 1
            for (int ch = w; ch < nch; ch += FX_NW) {
                const int i = ch * WAVE + lane, v = i < n ? u_at[i] - d0 : -1;
                const bool in = (unsigned)v < 64u;
                uint64_t same = __ballot(in);
#pragma unroll
                for (int bit = 0; bit < 6; ++bit) {
                    const uint64_t bal = __ballot((v >> bit) & 1);
                    same &= (v >> bit) & 1 ? bal : ~bal;
                }
                const int rank = (int)__popcll(same & lanemask_lt());
                if (in) {
                    u_rank[i] = rank;
                    if (rank == 0) h_cnt[ch * 64 + v] = (int)__popcll(same);
                }
            }
            __syncthreads();
            if (w == 0) {                                         // lane = row number: counts of the chunks to positions
                int sum = 0;
#pragma unroll 1
                for (int c = 0; c < nch; ++c) {
                    const int x = h_cnt[c * 64 + lane];
                    h_cnt[c * 64 + lane] = sum;
                    sum += x;
                }
                int inc = sum;
#pragma unroll
                for (int s = 1; s < 64; s <<= 1) {
                    const int o = __shfl_up(inc, s);
                    if (lane >= s) inc += o;
                }
                if (d0 + lane < D) s_start[d0 + lane] = (uint16_t)(placed + inc - sum);
                placed += __shfl(inc, 63);
            }
            __syncthreads();
#pragma unroll 1
            for (int i = t; i < n; i += FX_T) {
                const int num = u_at[i];
                if ((unsigned)(num - d0) >= 64u) continue;
                const int at = (int)s_start[num] + h_cnt[(i >> 6) * 64 + num - d0] + u_rank[i], k = u_k[i];
                const uint32_t row = u_r[i];
                int x1, x2, x3;
                decode_f64(p, row, x1, x2, x3);
                const bool is_head = (s_heads[i >> 6] >> (i & 63)) & 1;
                a.w.rec[k - k0] = is_head ? make_int2(x1, x3) : make_int2(-1, -1);
                if (is_head) s_row[num] = row;
                s_k[at] = k; s_bag[at] = bag_find(k);
            }
            if (d0 + 64 < D) {
                __syncthreads();
                for (int x = t; x < nch * 64; x += FX_T) h_cnt[x] = 0;
                __syncthreads();
            }
        }
        if (t == 0) s_start[D] = (uint16_t)n;
        __syncthreads();
        for (int d0 = 0; d0 < D; d0 += d.TP) {
            const bool final = last && d0 + d.TP >= D;
            tile(d0, min(d.TP, D - d0), final);
            in_part = !(final && d.S == 1);
        }
    };

    // scan: wave w looks at 256 consecutive positions of a round, the list stays in the order of the positions
    int cnt = 0, parity = 0;
    bool done = false;                                            // the slice has been finished (S == 1)
    uint32_t nrow_[4];
    int nsl[4];
    auto fetch = [&](int base) {                                  // a round ahead
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = min(base + w * 256 + q * 64 + lane, k_hi - 1);
            nrow_[q] = (uint32_t)a.indices[k];
            nsl[q] = a.slot ? a.slot[k] : -1;
        }
    };
    if (k_lo < k_hi) fetch(k_lo);
    if (search) load_offsets();
    fetch_bm(0);
    for (int base = k_lo; base < k_hi; base += FX_ROUND, parity ^= 1) {
        uint32_t row[4];
        int sl[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) { row[q] = nrow_[q]; sl[q] = nsl[q]; }
        if (base + FX_ROUND < k_hi) fetch(base + FX_ROUND);
        uint64_t m[4];
        int mine = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = base + w * 256 + q * 64 + lane;
            m[q] = __ballot(k < k_hi && sl[q] < 0 && select_digit_f64(p, 1, (double)row[q]) == (double)i2);
            if (sl[q] >= 0 && i2 == 0 && k < k_hi) a.w.rec[k - k0] = make_int2(-1, -1);    // a cached position stands for no row
            mine += __popcll(m[q]);
        }
        if (lane == 0) s_cnt[parity][w] = mine;
        __syncthreads();
        int at = cnt;
#pragma unroll
        for (int q = 0; q < FX_NW; ++q) {
            const int x = s_cnt[parity][q];
            if (q < w) at += x;
            cnt += x;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((m[q] >> lane) & 1) {
                const int pos = at + __popcll(m[q] & lanemask_lt());
                u_k[pos] = base + w * 256 + q * 64 + lane;
                u_r[pos] = row[q];
            }
            at += __popcll(m[q]);
        }
        const bool last = base + FX_ROUND >= k_hi;
        // (a pass that starts inside a segment starts at a piece)
        const bool end = last || (!ONE && (base - k_lo + FX_ROUND) % d.piece == 0);
        if (cnt > 0 && (end || cnt > FX_CAP - FX_ROUND)) {        // uniform
            __syncthreads();
            work(cnt, last && fin);
            if (last) done = d.S == 1 && fin;
            cnt = 0;
        }
    }
    if (!done) {                                                  // no positions, or none in the last window
        __syncthreads();
        if (d.S > 1 || !fin) {
            if (!in_part)
                for (int x = t; x < p.sB; x += FX_T) part[x] = 0.f;
        } else if (in_part) {
            for (int x = t; x < p.sB; x += FX_T) dst2[x] = fmaf(a.mul, part[x], src2[x]);
        } else if (dst2 != src2) {
            for (int x = t; x < p.sB; x += FX_T) dst2[x] = src2[x];
        }
    }
}

// Workgroups [0, m1): slices of the first core, [m1, m1 + m3): of the third; the rest (a.fold): sums of the parts of the second.
template <bool ONE>
__global__ __launch_bounds__(WG) void flex_sum_kernel(FlexArgs a)
{
    constexpr int CAP = FX_ROUND + 512, NF = 8;
    __shared__ int s_list[CAP];
    __shared__ float s_acc[1024];
    __shared__ __align__(16) float s_red[WG * 4];
    __shared__ int s_cnt[2][NWAVE];
    const Params &p = a.p;
    const int k0 = ONE ? 0 : a.k0, k1 = ONE ? a.L : a.k1;
    const bool fin = ONE || a.fin;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int b = blockIdx.x;
    if (b >= p.m1 + p.m3) {
        const int64_t n = (int64_t)p.m2 * p.sB;
        const int parts = (k1 - k0 + a.d.seg - 1) / a.d.seg;
        const bool more = k0 >= a.d.seg;                          // earlier segments are in acc
        float *acc = a.w.acc + (size_t)p.m1 * p.sA + (size_t)p.m3 * p.sC;
        for (int64_t i = (int64_t)(b - p.m1 - p.m3) * WG + t; i < n; i += (int64_t)(gridDim.x - p.m1 - p.m3) * WG) {
            float s = a.w.part[i];
            if (more) s = acc[i] + s;
            for (int q = 1; q < parts; ++q) s += a.w.part[q * n + i];
            if (fin) a.dst[1][i] = fmaf(a.mul, s, a.src[1][i]);
            else acc[i] = s;
        }
        return;
    }
    const bool third = b >= p.m1;
    const int s = third ? b - p.m1 : b, width = third ? p.sC : p.sA;
    const float *buf = third ? a.w.cbuf : a.w.pbuf;
    const float *src = (third ? a.src[2] : a.src[0]) + (size_t)s * width;
    float *dst = (third ? a.dst[2] : a.dst[0]) + (size_t)s * width;
    float *acc = a.w.acc + (third ? (size_t)p.m1 * p.sA : 0) + (size_t)s * width;
    const int n = k1 - k0;                                        // positions of the pass
    bool any = !ONE && !a.first;
    if (any)                                                      // (added to by the threads that add_up's barriers order)
        for (int x = t; x < width; x += WG) s_acc[x] = acc[x];

    // adds the listed rows up: a power of two of lanes per row, the groups of lanes take every ng-th entry
    auto add_up = [&](int n, auto vw) {
        constexpr int VW = decltype(vw)::value;
        const int nv = width / VW;
        int lp = 1, sh = 0;
        while (lp < nv && lp < WG) { lp <<= 1; ++sh; }
        const int f = t & (lp - 1), g = t >> sh, ng = WG >> sh;
        for (int c0 = 0; c0 < nv; c0 += lp) {                     // uniform
            const bool on = c0 + f < nv;
            const float *bf = buf + (on ? VW * (c0 + f) : 0);
            float sum[VW] = {};
            for (int i = g; i < n; i += NF * ng) {
                float x[NF][VW];
#pragma unroll
                for (int q = 0; q < NF; ++q) load_vec<VW>(bf + (size_t)s_list[min(i + q * ng, n - 1)] * width, x[q]);
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    if (i + q * ng < n) {
#pragma unroll
                        for (int v = 0; v < VW; ++v) sum[v] += x[q][v];
                    }
            }
            store_vec<VW>(s_red + t * VW, sum);
            __syncthreads();
            if (g == 0 && on) {
                float tot[VW] = {};
                for (int q = 0; q < ng; ++q) {
                    float x[VW];
                    load_vec<VW>(s_red + (q * lp + f) * VW, x);
#pragma unroll
                    for (int v = 0; v < VW; ++v) tot[v] += x[v];
                }
#pragma unroll
                for (int v = 0; v < VW; ++v) {
                    float *q = s_acc + VW * (c0 + f) + v;
                    *q = any ? *q + tot[v] : tot[v];
                }
            }
            __syncthreads();
        }
        any = true;
    };

    int cnt = 0, parity = 0;
    for (int base = 0; base < n; base += FX_ROUND, parity ^= 1) {
        int2 rc[FX_ROUND / WG];
#pragma unroll
        for (int q = 0; q < FX_ROUND / WG; ++q) rc[q] = a.w.rec[min(base + w * (FX_ROUND / NWAVE) + q * 64 + lane, n - 1)];
        uint64_t m[FX_ROUND / WG];
        int mine = 0;
#pragma unroll
        for (int q = 0; q < FX_ROUND / WG; ++q) {
            m[q] = __ballot(base + w * (FX_ROUND / NWAVE) + q * 64 + lane < n && (third ? rc[q].y : rc[q].x) == s);
            mine += __popcll(m[q]);
        }
        if (lane == 0) s_cnt[parity][w] = mine;
        __syncthreads();
        int at = cnt;
#pragma unroll
        for (int q = 0; q < NWAVE; ++q) {
            const int x = s_cnt[parity][q];
            if (q < w) at += x;
            cnt += x;
        }
#pragma unroll
        for (int q = 0; q < FX_ROUND / WG; ++q) {
            if ((m[q] >> lane) & 1) s_list[at + __popcll(m[q] & lanemask_lt())] = base + w * (FX_ROUND / NWAVE) + q * 64 + lane;
            at += __popcll(m[q]);
        }
        bool end = base + FX_ROUND >= n;
        if constexpr (!ONE) {
            const int in_seg = (k0 + base) % a.d.seg + FX_ROUND;  // (the segment's length is a multiple of the round's)
            end |= a.d.piece >= a.d.seg ? (k0 + base + FX_ROUND) % a.d.piece == 0 : in_seg == a.d.seg || in_seg % a.d.piece == 0;
        }
        if (cnt > 0 && (end || cnt > CAP - FX_ROUND)) {           // uniform
            __syncthreads();
            if ((width & 3) == 0) add_up(cnt, std::integral_constant<int, 4>{});
            else add_up(cnt, std::integral_constant<int, 1>{});
            cnt = 0;
        }
    }
    if (!fin) {                                                   // (-0 + x is x, whatever x is)
        __syncthreads();
        for (int x = t; x < width; x += WG) acc[x] = any ? s_acc[x] : -0.f;
    } else if (any) {
        if constexpr (!ONE) __syncthreads();
        for (int x = t; x < width; x += WG) {
            const float v = s_acc[x];
            dst[x] = !ONE && v == 0.f ? src[x] : fmaf(a.mul, v, src[x]);   // (a slice without positions in any of several passes: copied)
        }
    } else if (dst != src) {
        for (int x = t; x < width; x += WG) dst[x] = src[x];
    }
}

// ---- forward -------------------------------------------------------------------------------------------------------
// A wave per bag.  J rows j1 at a time, V columns per lane: T0[j1][c] = sum_a A[j1][a] Bm[a][c] in registers (A through
// scalar loads), to the wave's part of LDS; then lane (part, j) adds every parts-th value of b of output j.
// NCH: the rank R1 in eights where it is a multiple and one turn over j1 and over the columns does (J == n1, cols <= 64 V):
// then every load of a position is in flight at once.  0: whatever the shape.
template <int J, int V, int NCH>
__global__ __launch_bounds__(WG) void flex_fwd_kernel(Params p, const float *__restrict__ G1, const float *__restrict__ G2,
                                                      const float *__restrict__ G3, const int64_t *__restrict__ indices,
                                                      const int64_t *__restrict__ offsets, int n_bags, const float *__restrict__ alpha,
                                                      CacheDev cache, float *__restrict__ out)
{
    extern __shared__ __align__(16) float fx_t[];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n1 = p.n1, n3 = p.n3, R1 = p.R1, R2 = p.R2, N = p.N, cols = p.cols;
    float *T = fx_t + (size_t)wv * n1 * cols;
    const int bag = blockIdx.x * NWAVE + wv;
    if (bag >= n_bags) return;                                    // (no barrier below: the waves are independent)
    const int k0 = offsets ? (int)offsets[bag] : bag, k1 = offsets ? (int)offsets[bag + 1] : bag + 1;
    int parts = 1;
    if ((N & (N - 1)) == 0)
        while (2 * parts * N <= WAVE) parts <<= 1;
    const int part = parts > 1 ? lane / N : 0, j0 = parts > 1 ? lane % N : lane;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};                          // outputs j0, j0 + 64, ... (N <= 256)
    int oq[4], o3[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int j = min(j0 + 64 * u, N - 1);
        oq[u] = j / n3;
        o3[u] = j - oq[u] * n3;
    }
    const int nu = parts > 1 ? 1 : (N + 63) / 64;
    for (int kb = k0; kb < k1; kb += WAVE) {
        const int nb = min(WAVE, k1 - kb);
        const uint32_t prow = lane < nb ? (uint32_t)indices[kb + lane] : 0u;
        const float pw = lane < nb && alpha ? alpha[kb + lane] : 1.f;
        const int psl = cache.K && lane < nb ? cache_probe(cache, prow) : -1;
        for (int j = 0; j < nb; ++j) {
            const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)prow, j);
            const float wgt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pw), j));
            const int sl = __builtin_amdgcn_readlane(psl, j);
            if (sl >= 0) {
                if (part == 0)
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (j0 + 64 * u < N) acc[u] = fmaf(wgt, cache.rows[(size_t)sl * N + j0 + 64 * u], acc[u]);
                continue;
            }
            int i1, i2, i3;
            decode(p, row, i1, i2, i3);
            const float *A = G1 + (size_t)i1 * p.sA, *Bm = G2 + (size_t)i2 * p.sB, *C = G3 + (size_t)i3 * p.sC;
            // the third core's values of the second product, on their way while the first one runs (as many as fit 16 registers)
            float cpre[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) cpre[q] = C[min(part + q * parts, R2 - 1) * n3 + o3[0]];
            if constexpr (NCH > 0) {
                constexpr int RR = 8 * NCH;
                const int c0 = min(lane * V, cols - V);            // (lanes without columns: any, not stored)
                float bv[RR][V], t0[J][V];
#pragma unroll
                for (int x = 0; x < RR; ++x) load_vec<V>(Bm + x * cols + c0, bv[x]);
#pragma unroll
                for (int q = 0; q < J; ++q)
#pragma unroll
                    for (int v = 0; v < V; ++v) t0[q][v] = 0.f;
#pragma unroll
                for (int x = 0; x < RR; ++x)
#pragma unroll
                    for (int q = 0; q < J; ++q) {
                        const float av = A[q * RR + x];
#pragma unroll
                        for (int v = 0; v < V; ++v) t0[q][v] = fmaf(av, bv[x][v], t0[q][v]);
                    }
                if (lane * V < cols)
#pragma unroll
                    for (int q = 0; q < J; ++q) store_vec<V>(T + q * cols + c0, t0[q]);
            } else {
                for (int jc = 0; jc < n1; jc += J)
                    for (int c0 = lane * V; c0 < cols; c0 += WAVE * V) {
                        float t0[J][V];
#pragma unroll
                        for (int q = 0; q < J; ++q)
#pragma unroll
                            for (int v = 0; v < V; ++v) t0[q][v] = 0.f;
                        const float *B = Bm + c0;
                        int a = 0;
                        for (; a + 8 <= R1; a += 8) {                  // eight row loads in flight
                            float bv[8][V];
#pragma unroll
                            for (int x = 0; x < 8; ++x) load_vec<V>(B + (a + x) * cols, bv[x]);
#pragma unroll
                            for (int x = 0; x < 8; ++x)
#pragma unroll
                                for (int q = 0; q < J; ++q) {
                                    const float av = A[min(jc + q, n1 - 1) * R1 + a + x];
#pragma unroll
                                    for (int v = 0; v < V; ++v) t0[q][v] = fmaf(av, bv[x][v], t0[q][v]);
                                }
                        }
                        for (; a < R1; ++a) {
                            float bv[V];
                            load_vec<V>(B + a * cols, bv);
#pragma unroll
                            for (int q = 0; q < J; ++q) {
                                const float av = A[min(jc + q, n1 - 1) * R1 + a];
#pragma unroll
                                for (int v = 0; v < V; ++v) t0[q][v] = fmaf(av, bv[v], t0[q][v]);
                            }
                        }
#pragma unroll
                        for (int q = 0; q < J; ++q)
                            if (jc + q < n1) store_vec<V>(T + (jc + q) * cols + c0, t0[q]);
                    }
            }
            __builtin_amdgcn_wave_barrier();                       // (LDS of one wave is in order: only the compiler has to keep it)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nu) {                                      // uniform
                    float s = 0.f;
                    const float *Tq = T + oq[u] * R2, *Cq = C + o3[u];
                    int b = part;
                    if (u == 0) {
                        float tq[16];                              // (read at once, picked afterwards)
#pragma unroll
                        for (int q = 0; q < 16; ++q) tq[q] = Tq[min(part + q * parts, R2 - 1)];
#pragma unroll
                        for (int q = 0; q < 16; ++q, b += parts) s = b < R2 ? fmaf(tq[q], cpre[q], s) : s;
                    }
                    for (; b + 7 * parts < R2; b += 8 * parts) {   // eight loads in flight
                        float x[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) x[q] = Cq[(b + q * parts) * n3];
#pragma unroll
                        for (int q = 0; q < 8; ++q) s = fmaf(Tq[b + q * parts], x[q], s);
                    }
                    for (; b < R2; b += parts) s = fmaf(Tq[b], Cq[b * n3], s);
                    acc[u] = fmaf(wgt, s, acc[u]);
                }
            __builtin_amdgcn_wave_barrier();
        }
    }
    for (int s = N; s < parts * N; s <<= 1) acc[0] += __shfl_xor(acc[0], s);
    if (part == 0)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j0 + 64 * u < N) out[(size_t)bag * N + j0 + 64 * u] = acc[u];
}

// ---- host side -------------------------------------------------------------------------------------------------------

// columns per lane of the forward pass: no more than leave every lane some, and whole vectors
static inline int flex_fwd_v(const Params &p) { return p.cols > 128 && p.cols % 4 == 0 ? 4 : (p.cols > 64 && p.cols % 2 == 0 ? 2 : 1); }
static inline int flex_fwd_j(const Params &p) { return p.n1 <= 2 ? 2 : 4; }

// One turn and the rank in eights (see flex_fwd_kernel): ahead of the plain kernel for all of 25 such shapes.  4,096 bags of one
// position / 64 of 60, eight rows at a time, this, plain: (4,4,4) at rank 16 11.0 / 151, 7.4 / 64 and 10.6 / 171 us, (2,4,4) at 24
// 10.7 / 136, 9.4 / 74, 12.7 / 239, (4,4,4) at 8 -, 6.5 / 51, 7.8 / 102, (4,3,4) at (32,16) 14.2 / 211, 9.0 / 104, 13.5 / 269.
static inline bool flex_fwd_one_turn(const Params &p)
{
    const int V = flex_fwd_v(p);
    return p.n1 == flex_fwd_j(p) && p.cols <= WAVE * V && p.cols % V == 0 && p.R1 % 8 == 0 && p.R1 <= 32;
}

// Is the wave per bag ahead of the plain kernel, which gives a bag four waves and a position three barriers?  The wave pays for
// turns over rows j1 that are not all there, for lanes without columns and, eight loads or one at a time, for ranks and outputs
// off its steps; the plain kernel for its rounds of 256 values and one load after the other along the ranks.  What a position
// takes is estimated for both, in units of 10 ns, from timings of 100 shapes in bags of 60 positions (the estimates are off by 9 and 5 % at the
// median).  Few bags, many short ones and many single ones all come out the same way; wave / plain, 64 bags of 60: (4,4,8) at
// rank 64 657 / 1,966 us, (5,3,7) at (17,33)
// 469 / 293, (6,6,6) at 7 272 / 97, (16,1,16) at (64,3) 1,269 / 313.  The kernel so chosen was the slower one by more than 10 %, and
// by up to 31 %, for three of the 100.
static inline bool flex_fwd_pays(const Params &p)
{
    if (flex_fwd_one_turn(p)) return true;
    auto up = [](int a, int b) { return (a + b - 1) / b; };
    auto trips = [](int n) { return n > 0 ? n / 8 + n % 8 : 0; };              // (the last ones one at a time)
    const int V = flex_fwd_v(p), J = flex_fwd_j(p), turns = up(p.n1, J) * up(p.cols, WAVE * V);
    int parts = 1;
    if ((p.N & (p.N - 1)) == 0)
        while (2 * parts * p.N <= WAVE) parts <<= 1;
    const int per = up(p.R2, parts), outs = parts > 1 ? 1 : up(p.N, WAVE);     // values of b per lane, outputs per lane
    const double wave = 90 + turns * (44 + 4.5 * trips(p.R1) + 0.64 * p.R1 * J * V) + 5.6 * (trips(per - 16) + (outs - 1) * trips(per)) + 1.7 * outs * per;
    const double plain = 55 + 8.3 * up(p.n1 * p.cols, WG) * p.R1 + 5.3 * p.R2;
    return wave <= plain;
}

static inline size_t flex_fwd_lds(const Params &p) { return (size_t)NWAVE * p.n1 * p.cols * sizeof(float); }

static inline void flex_fwd(const Params &p, const float *G1, const float *G2, const float *G3, const int64_t *idx, const int64_t *off,
                            int n_bags, const float *alpha, const CacheDev &cd, float *out, hipStream_t st)
{
    const dim3 grid((n_bags + NWAVE - 1) / NWAVE), wg(WG);
    const size_t lds = flex_fwd_lds(p);
    const int V = flex_fwd_v(p);
    const int J = flex_fwd_j(p);
    auto launch = [&](auto j, auto v) {
        auto go = [&](auto nch) {
            hipLaunchKernelGGL((flex_fwd_kernel<decltype(j)::value, decltype(v)::value, decltype(nch)::value>), grid, wg, lds, st, p, G1, G2, G3,
                               idx, off, n_bags, alpha, cd, out);
        };
        switch (flex_fwd_one_turn(p) ? p.R1 / 8 : 0) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        default: go(std::integral_constant<int, 0>{});
        }
    };
    auto with_v = [&](auto j) {
        if (V == 4) launch(j, std::integral_constant<int, 4>{});
        else if (V == 2) launch(j, std::integral_constant<int, 2>{});
        else launch(j, std::integral_constant<int, 1>{});
    };
    if (J == 2) with_v(std::integral_constant<int, 2>{});
    else with_v(std::integral_constant<int, 4>{});
}

// pass: what flex_pass says for the workspace that a.w lies in
static inline hipError_t flex_bwd(FlexArgs a, int64_t pass, hipStream_t st)
{
    const Params &p = a.p;
    const bool v4 = p.n3 == 4 && ((p.R1 | p.R2) & 3) == 0;
    const bool one = a.L <= a.d.whole;
    void (*const g2)(FlexArgs) = v4 ? (one ? flex_g2_kernel<true, true> : flex_g2_kernel<true, false>) : (one ? flex_g2_kernel<false, true> : flex_g2_kernel<false, false>);
    static OncePerDevice once[4];
    hipError_t e = allow_dynamic_lds(once[2 * v4 + one], (const void *)g2, FX_MAX_LDS);
    if (e != hipSuccess) return e;
    const int fin = a.d.S > 1 ? (int)(((int64_t)p.m2 * p.sB + 4 * WG - 1) / (4 * WG)) : 0;
    const size_t lds = (size_t)a.d.lds_floats * sizeof(float);
    for (int64_t k = 0; k < a.L; k = a.k1) {
        const int64_t seg_end = (k / a.d.seg + 1) * a.d.seg;
        int64_t end = k + pass;
        if (pass < a.d.seg && end > seg_end) end = seg_end;
        if (end > a.L) end = a.L;
        a.k0 = (int)k;
        a.k1 = (int)end;
        a.cont = k % a.d.seg != 0;
        a.first = k == 0;
        a.fin = end == a.L;
        a.fold = a.d.S > 1 && (a.fin || end % a.d.seg == 0);
        const dim3 grid(p.m2 * (int)((end - k + a.d.seg - 1) / a.d.seg)), wg(FX_T);
        hipLaunchKernelGGL(g2, grid, wg, lds, st, a);
        hipLaunchKernelGGL(one ? flex_sum_kernel<true> : flex_sum_kernel<false>, dim3(p.m1 + p.m3 + (!a.fold ? 0 : fin < 4096 ? fin : 4096)), dim3(WG), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace tt
