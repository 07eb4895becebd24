// Forward pass over the distinct rows of a batch, without T0 and without a cache (tt_emb_fwd_rows): five launches.
//
//   rw_count / rw_scatter   (tt_rows.h) positions grouped by their second digit
//   rf_group_kernel         equal rows of a window of RF_WIN positions of a slice meet in a hash table in LDS; the distinct ones are
//                           numbered, every position is told the number of its row
//   rf_rows_kernel          tiles of distinct rows of one slice: T0 = A Bm (Eq. 3, first product) on the matrix cores, one j2
//                           at a time, then the row itself (second product)
//   rw_pool_kernel          (tt_rows_pass.h) a wave per bag, or a part of one, adds the weighted rows of its positions
//
// The number of a row decides where it is kept and which tile it is in, nothing else; results repeat bit for bit.
// (One workgroup per slice that looks through all indices, in place of the first three launches: 6 against 14 us at 4,096
// positions, where the wave per bag is ahead anyway, 31 against 17 at 73,000, with the hot row's slice the last to finish.)
#pragma once

#include "tt_rows_pass.h"

namespace tt {

constexpr int RF_WIN = RW_T;                     // positions of a window: one per thread; a row that two windows share is computed twice
constexpr int64_t RF_SHORT_L = 131072;           // up to here short tiles in the counting pass
constexpr size_t RF_MAX_BYTES = (size_t)1 << 30; // scratch memory that a call is worth (tt_emb_fwd_rows_pays)
// Positions of a call, fewer than this: up to there a tile past the last position is still an int, and a launch with 1,024 threads
// per window of at least 512 positions, or per slice, has fewer than the 2^32 threads that a grid can have.
constexpr int64_t RF_MAX_L = (1ll << 31) - (1ll << 20);
static_assert(RF_MAX_L + RW_TILE <= (1ll << 31) && (RF_MAX_L / RF_WIN + RW_MAX_M2) * 1024 < (1ll << 32), "what the limit is for");

static inline int rf_tile(int64_t L) { return L < RF_SHORT_L ? RW_TILE_SHORT : RW_TILE; }

// the parts of RowsWs that are used here
static inline RowsWs rf_ws_layout(void *ws, const Params &p, int64_t L)
{
    RowsWs w{};
    char *base = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *q = base ? base + off : nullptr; off += align256(bytes); return q; };
    const size_t n = L > 0 ? (size_t)L : 1, nw = (size_t)rw_windows_of(p, L, RF_WIN);
    w.hist = (uint32_t *)take((size_t)((n + rf_tile(L) - 1) / rf_tile(L)) * ((p.m2 + 3) & ~3) * 4);
    w.lk = (uint32_t *)take(n * 4);
    w.lrow = (uint32_t *)take(n * 4);
    w.goff = (int *)take(((size_t)p.m2 + 1) * 4);
    w.inv = (int *)take(n * 4);
    w.rec = (int4 *)take(n * 16);
    w.wd = (int *)take(nw * 4);
    w.wfirst = (int *)take(nw * 4);
    w.wslice = (int *)take(nw * 4);
    w.nwin = (int *)take(4);
    w.rows = (float *)take(n * p.N * 4);
    w.bytes = off;
    return w;
}

__global__ __launch_bounds__(RW_T) void rf_group_kernel(Params p, RowsWs ws)
{
    constexpr int HASH = 2 * RF_WIN;
    __shared__ uint32_t h_row[HASH];
    __shared__ int h_num[HASH], s_tmp[RW_NW], s_win[2];
    __shared__ int s_distinct;
    const int t = threadIdx.x;
    for (int x = t; x < HASH; x += RW_T) h_row[x] = ~0u;
    if (t == 0) s_distinct = 0;
    if (!rw_find_window(p, RF_WIN, ws, s_tmp, s_win)) return;       // uniform
    __syncthreads();
    const int slice = s_win[0], first = ws.goff[slice] + s_win[1] * RF_WIN, n = min(RF_WIN, ws.goff[slice + 1] - first);
    const uint32_t row = ws.lrow[first + min(t, n - 1)], k = ws.lk[first + min(t, n - 1)];
    uint32_t h = cache_hash(row, HASH - 1), old;
    if (t < n) {
        for (;;) {                                                 // ends: at most RF_WIN rows in twice as many places
            old = atomicCAS(&h_row[h], ~0u, row);
            if (old == ~0u || old == row) break;
            h = (h + 1) & (HASH - 1);
        }
        if (old == ~0u) {
            const int num = first + atomicAdd(&s_distinct, 1);
            int i1, i2, i3;
            decode_f64(p, row, i1, i2, i3);
            h_num[h] = num;
            ws.rec[num] = make_int4(i1, i3, 0, 1);
        }
    }
    __syncthreads();
    if (t < n) ws.inv[k] = h_num[h];
    if (t == 0) {
        ws.wd[blockIdx.x] = s_distinct;
        ws.wfirst[blockIdx.x] = first;
        ws.wslice[blockIdx.x] = slice;
    }
}

// Sums over 8 (4) neighbouring lanes of 16 (8) values each, two of which a lane ends with.  In every step a lane keeps half of
// its values and takes those of its partner on top, through DPP: within 8 lanes l and 7 - l, then l and l ^ 2, then l and l ^ 1.
// (By __shfl_xor of everything, 48 values per lane went through LDS.)
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141;

template <int NV, int CTRL, int BIT, int N>
__device__ __forceinline__ void dpp_halve(float (&v)[N], int lane)           // of v[0 .. NV), v[0 .. NV / 2) hold the sums kept
{
    const bool up = (lane & BIT) != 0;
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) {
        const float keep = up ? v[i + NV / 2] : v[i], give = up ? v[i] : v[i + NV / 2];
        v[i] = keep + dpp_of<CTRL>(give);
    }
}

template <typename C>
struct RfCols {
    static constexpr int NW = C::sB * 4 > 32768 ? 8 : 4;   // waves per workgroup: more where the slice leaves room for one only
    static constexpr int EU = C::R >= 64 ? 2 : 4;          // waves per SIMD that the slice leaves room for
    static constexpr int EB = 32 / C::N1;            // distinct rows of a block: 32 stacked rows (row, j1)
    static constexpr int PARTS = 128 / EB / NW;      // workgroups that share a window's blocks
    static_assert(PARTS * NW * WAVE <= 1024, "threads per window: see RF_MAX_L");
    static constexpr int NBQ = WAVE / EB;            // lanes per row in the second product: a part of b each
    static constexpr int BQ = C::R / NBQ;            // values of b per lane
    static constexpr int KH = C::R / 2;              // steps of the first product: k values per half of the wave
    static constexpr int CB = C::R / 32;             // 32-column blocks
    static constexpr int LDT = C::R + 2;             // row stride of T0 in LDS
    static constexpr int NV = 4 * C::N1;             // values of a row per j2
    static constexpr size_t LDS = (size_t)(C::sB + NW * 32 * LDT) * sizeof(float);
    static_assert((NBQ == 8 && NV == 16) || (NBQ == 4 && NV == 8), "the sums over the lanes of a row are written for these");
};

// A workgroup has the slice of a window in LDS; its waves take blocks of 32 stacked rows (EB distinct rows) each on their own:
// the first core's rows straight from memory as the first operand, T0 of one j2 through a part of LDS of the wave's own to the
// second product.  So a row's slices are read once and nothing but the slice is waited for together.
// 73,000 positions with 23,000 distinct rows, (4,4,4) at rank 32: 21 us, of which 5 are matrix products at their peak rate and 12
// are what a single block takes (launch, four round trips, four times two products).  Tried: tiles of 128 stacked rows per
// workgroup with barriers on either side of every j2 (25 us; a single tile 17), a wave per j2 with its part of the slice in
// registers, which reads a row's slices n2 times (23 us; a single block 9, but every row different 57 against 43), the slice's
// operands of the next j2 read ahead of the products (no change at rank 32, spills at 64).
template <typename C>
__global__ __launch_bounds__(RfCols<C>::NW *WAVE) __attribute__((amdgpu_waves_per_eu(RfCols<C>::EU, RfCols<C>::EU))) void rf_rows_kernel(Params p, const float *__restrict__ G1, const float *__restrict__ G2,
                                                                      const float *__restrict__ G3, int L, RowsWs ws)
{
    using F = RfCols<C>;
    constexpr int N1 = C::N1, N2 = C::N2, R = C::R, COLS = C::COLS, EB = F::EB, KH = F::KH, CB = F::CB, LDT = F::LDT, NV = F::NV, NBQ = F::NBQ;
    constexpr int NT = F::NW * WAVE, STEP = F::PARTS * F::NW * EB;
    extern __shared__ __align__(16) float rf_slice[];                         // [R][COLS], then [NW][32][LDT]
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ln = lane & 31, kh = lane >> 5, win = blockIdx.x / F::PARTS, part = blockIdx.x % F::PARTS;
    if (win >= *ws.nwin) return;                                              // uniform
    const int i2 = ws.wslice[win], first = ws.wfirst[win], D = ws.wd[win];
    // (Never so.  But it has all three loaded by here: the compiler moves two of them below the next branch otherwise, which is a round
    // trip of its own: 73,600 positions, (4,4,4) at rank 32, 41.1 us with this line, 41.4 without.)
    if ((unsigned)i2 >= (unsigned)p.m2 || first < 0 || D < 0 || first > L - D) return;
    if (part * F::NW * EB >= D) return;                                       // uniform
    float *T = rf_slice + C::sB + w * 32 * LDT;
    const int ea = ln / N1, j1 = ln % N1;                                     // row and j1 of this lane in the first product
    const int ee = lane / NBQ, bq = lane % NBQ;                               // row and part of b in the second one
    int d0 = (part * F::NW + w) * EB, i1, i3;
    auto records = [&]() __attribute__((always_inline)) {
        i1 = ws.rec[first + min(d0 + ea, D - 1)].x;
        i3 = ws.rec[first + min(d0 + ee, D - 1)].y;
    };
    float areg[KH], cv[F::BQ][4];
    auto fetch = [&]() __attribute__((always_inline)) {
        const float *Ap = G1 + (size_t)i1 * C::sA + j1 * R + kh * KH;         // step s of the first product covers k = kh KH + s
#pragma unroll
        for (int q = 0; q < KH / 4; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(Ap + 4 * q);
            areg[4 * q + 0] = x.x; areg[4 * q + 1] = x.y; areg[4 * q + 2] = x.z; areg[4 * q + 3] = x.w;
        }
        const float4 *Cp = reinterpret_cast<const float4 *>(G3 + (size_t)i3 * C::sC) + bq;   // (the NBQ lanes of a row read neighbouring rows of G3[i3])
#pragma unroll
        for (int i = 0; i < F::BQ; ++i) {
            const float4 v = Cp[i * NBQ];
            cv[i][0] = v.x; cv[i][1] = v.y; cv[i][2] = v.z; cv[i][3] = v.w;
        }
    };
    records();
    {
        constexpr int NS = C::sB / 4 / NT;
        static_assert(NS * 4 * NT == C::sB, "whole float4 per thread");
        const float4 *src = reinterpret_cast<const float4 *>(G2 + (size_t)i2 * C::sB);
        float4 v[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) v[q] = src[q * NT + threadIdx.x];
        fetch();                                                              // (before the barrier: all of it in flight together)
#pragma unroll
        for (int q = 0; q < NS; ++q) reinterpret_cast<float4 *>(rf_slice)[q * NT + threadIdx.x] = v[q];
    }
    __syncthreads();
    const float *B0 = rf_slice + kh * KH * COLS + ln;
    for (; d0 < D; d0 += STEP) {                                              // uniform in the wave
        float *out = ws.rows + (size_t)(first + d0 + ee) * C::N;
        const bool on = d0 + ee < D;
        if (d0 + STEP < D) {
            d0 += STEP;
            records();                                                        // of the next block
            d0 -= STEP;
        }
#pragma unroll 1
        for (int j2 = 0; j2 < N2; ++j2) {
            const float *B = B0 + j2 * R;
            mfma16_t acc[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
#pragma unroll
            for (int s = 0; s < KH; ++s)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(areg[s], B[s * COLS + 32 * cb], acc[cb], 0, 0, 0);
            // register r of lane (kh, ln) is row 8 (r / 4) + 4 kh + r % 4, column ln of its 32 x 32 block
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) T[(8 * (r / 4) + 4 * kh + r % 4) * LDT + 32 * cb + ln] = acc[cb][r];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");            // (LDS of one wave is in order: only the compiler has to keep it)
            __builtin_amdgcn_wave_barrier();
            float o[NV];
#pragma unroll
            for (int j = 0; j < NV; ++j) o[j] = 0.f;
#pragma unroll
            for (int i = 0; i < F::BQ; ++i)
#pragma unroll
                for (int j = 0; j < N1; ++j) {
                    const float tv = T[(ee * N1 + j) * LDT + i * NBQ + bq];
#pragma unroll
                    for (int x = 0; x < 4; ++x) o[4 * j + x] = fmaf(tv, cv[i][x], o[4 * j + x]);
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();                                  // the next j2 rewrites T
            int at = 0;                                                       // first of the two values that this lane ends with
            if constexpr (NBQ == 8) {
                dpp_halve<NV, DPP_HALF_MIRROR, 4>(o, lane);
                at = lane & 4 ? NV / 2 : 0;
            }
            constexpr int V2 = NBQ == 8 ? NV / 2 : NV;
            dpp_halve<V2, DPP_XOR2, 2>(o, lane);
            dpp_halve<V2 / 2, DPP_XOR1, 1>(o, lane);
            at += (lane & 2 ? V2 / 2 : 0) + (lane & 1 ? V2 / 4 : 0);
            if (on) *reinterpret_cast<float2 *>(out + ((at / 4) * N2 + j2) * 4 + at % 4) = make_float2(o[0], o[1]);
        }
        if (d0 + STEP < D) fetch();
    }
}

// ---- host side -------------------------------------------------------------------------------------------------------

template <typename C>
static inline hipError_t launch_rows_fwd(const Params &p, const float *G1, const float *G2, const float *G3, const int64_t *indices, int64_t L,
                                         const int64_t *off, int n_bags, const float *alpha, float *out, const RowsWs &ws, hipStream_t st)
{
    using F = RfCols<C>;
    static OncePerDevice once;
    hipError_t e = allow_dynamic_lds(once, (const void *)rf_rows_kernel<C>, F::LDS);
    if (e != hipSuccess) return e;
    const int nw = rw_windows_of(p, L, RF_WIN);
    const CacheDev none{nullptr, nullptr, 0, 0};
    rw_place(p, indices, (int)L, none, rf_tile(L), ws, st);
    hipLaunchKernelGGL(rf_group_kernel, dim3(nw), dim3(RW_T), 0, st, p, ws);
    hipLaunchKernelGGL(rf_rows_kernel<C>, dim3(nw * F::PARTS), dim3(F::NW * WAVE), F::LDS, st, p, G1, G2, G3, (int)L, ws);
    rw_pool<C::N>(ws.rows, ws.inv, nullptr, off, n_bags, L, alpha, out, st);
    return hipGetLastError();
}

static inline hipError_t rows_fwd(const Params &p, const float *G1, const float *G2, const float *G3, const int64_t *indices, int64_t L,
                                  const int64_t *off, int n_bags, const float *alpha, float *out, const RowsWs &ws, hipStream_t st)
{
    switch (fast_config(p)) {
    case 2: return launch_rows_fwd<Cfg224R32>(p, G1, G2, G3, indices, L, off, n_bags, alpha, out, ws, st);
    case 3: return launch_rows_fwd<Cfg224R64>(p, G1, G2, G3, indices, L, off, n_bags, alpha, out, ws, st);
    case 4: return launch_rows_fwd<Cfg444R32>(p, G1, G2, G3, indices, L, off, n_bags, alpha, out, ws, st);
    case 5: return launch_rows_fwd<Cfg444R64>(p, G1, G2, G3, indices, L, off, n_bags, alpha, out, ws, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace tt
