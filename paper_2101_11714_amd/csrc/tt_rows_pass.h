// Forward and backward pass over the distinct rows of a long index stream (the groups of tt_rows.h), with a kept T0.
//
// Forward (two launches).  rw_fwd_kernel: a workgroup takes a tile of distinct rows of one slice of the second core and one
// value of j2, computes their T0 = A Bm (Eq. 3, first product) on the matrix cores and their row from it, and copies T0 to
// all their positions; rw_pool_kernel: a wave per bag, or a part of one, adds the weighted rows of its positions.
// Backward (three launches).  rw_merge_kernel: the upstream gradients of a distinct row added up over its positions;
// rw_tile_kernel: Eq. 4's two large products over tiles of distinct rows,
//     dG2[i2][a][(j2,b)] += sum_rows A[(e,j1)][a] dT0'[(e,j1)][(j2,b)],   P[(e,j1)][a] = sum_(j2,b) dT0'[(e,j1)][(j2,b)] Bm[a][(j2,b)],
// with dT0'[(e,j1)][(j2,b)] = sum_j3 dY_e[(j1,j2)][j3] C_e[b][j3], as fp32 MFMA 32x32x2 products with operands in LDS, one j2
// at a time; rw_sum_kernel: the G1 gradient of a slice as the sum of its rows P, the G3 gradient as the sum of T0^T dY of
// its rows, and the parts of every slice of the second core, each finished with the SGD step or the "+=".
#pragma once

#include <type_traits>

#include "tt_rows.h"
#include "tt_bwd_owner.h"

namespace tt {

typedef float rw_f4 __attribute__((ext_vector_type(4)));   // what the store builtin takes

// ---- forward ---------------------------------------------------------------------------------------------------------

template <typename C, int ROWS_>
struct RfCfg {
    static constexpr int ROWS = ROWS_, TP = ROWS / C::N1;     // stacked rows / distinct rows per tile
    static constexpr int RB = ROWS / 32, WPR = NWAVE / RB;    // row blocks; waves that share one
    static constexpr int CBW = C::R / 32 / WPR;               // 32-column blocks per wave
    static constexpr int KH = C::R / 2;                       // k values per half of the wave
    static constexpr int LDT = C::R + 2;                      // row stride of the T0 block in LDS
    static constexpr int LDS_FLOATS = C::R * C::R > ROWS * LDT ? C::R * C::R : ROWS * LDT;
    static constexpr int NBQ = WG / TP < 16 ? WG / TP : 16;   // threads per row in the second product: a part of b each
    static constexpr int BQ = C::R / NBQ;                     // values of b per thread
    static constexpr bool EARLY_C = BQ <= 8;                  // fetch the third core's rows before the first product (if they fit the registers)
    static constexpr int GL = C::N1 * C::R / 4;               // threads per position when T0 is copied out
    static_assert(NWAVE % RB == 0 && C::R / 32 % WPR == 0 && CBW >= 1 && WG % TP == 0 && NBQ * TP == WG && GL <= WG, "tile layout");
};

template <typename C, int ROWS_>
__global__ __launch_bounds__(WG) void rw_fwd_kernel(Params p, const float *__restrict__ G1, const float *__restrict__ G2,
                                                    const float *__restrict__ G3, int L, const int4 *__restrict__ rec,
                                                    const int2 *__restrict__ gkb, const int *__restrict__ gu, const int4 *__restrict__ tiles,
                                                    const int *__restrict__ tile_base, float *__restrict__ rows_out, float *__restrict__ t0_out)
{
    using F = RfCfg<C, ROWS_>;
    constexpr int N1 = C::N1, N2 = C::N2, R = C::R, COLS = C::COLS, TP = F::TP, LDT = F::LDT;
    extern __shared__ __align__(16) float rf_lds[];
    __shared__ int s_k[RW_WIN];                                               // the tile's positions, and their rows in the tile
    __shared__ uint8_t s_e[RW_WIN];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int ln = lane & 31, kh = lane >> 5, rb = w % F::RB, cb0 = (w / F::RB) * F::CBW;
    const int j2 = blockIdx.x % N2, used = tile_base[p.m2];
    for (int tile = blockIdx.x / N2; tile < used; tile += gridDim.x / N2) {
        const int4 td = tiles[tile];
        const int i2 = td.x, u0 = td.y, n = td.z;
        if (n <= 0 || n > TP || (unsigned)i2 >= (unsigned)p.m2 || u0 < 0 || u0 + n > L) return;   // (no pre-pass wrote this)
        // this part of the slice, [R][R]: the loads first, the rows' records behind them
        constexpr int NB4 = R * R / 4 / WG;
        float4 bm[NB4];
        {
            const float *src = G2 + (size_t)i2 * C::sB + j2 * R;
#pragma unroll
            for (int q = 0; q < NB4; ++q) {
                const int i = q * WG + t, a = i / (R / 4), c4 = i % (R / 4);
                bm[q] = *reinterpret_cast<const float4 *>(src + a * COLS + 4 * c4);
            }
        }
        const int row = 32 * rb + ln, e = row / N1, j1 = row % N1;            // stacked first-core row of this lane
        const bool have = e < n;
        const int i1 = min(max(rec[u0 + (have ? e : 0)].x, 0), p.m1 - 1);
        const int ee = t / F::NBQ, bq = t % F::NBQ;                           // row and part of b of the second product
        const bool on = ee < n;
        const int i3 = min(max(rec[u0 + (on ? ee : 0)].y, 0), p.m3 - 1);
        const int4 r0 = rec[u0], r1 = rec[u0 + n - 1];
        const int E0 = r0.z, NE = min(r1.z + r1.w - E0, RW_WIN);              // the rows' positions are neighbours in gkb
        float4 cv[F::BQ];                                                     // (the NBQ lanes of a row read neighbouring rows of G3[i3])
        const float4 *Cp = reinterpret_cast<const float4 *>(G3 + (size_t)i3 * C::sC) + bq;
        if constexpr (F::EARLY_C) {
#pragma unroll
            for (int i = 0; i < F::BQ; ++i) cv[i] = Cp[i * F::NBQ];
        }
        // A operand: step s of the product covers k = kh KH + s (any order of k will do as long as both operands agree)
        float areg[F::KH];
        {
            const float *Ap = G1 + (size_t)i1 * C::sA + j1 * R + kh * F::KH;
#pragma unroll
            for (int q = 0; q < F::KH / 4; ++q) {
                const float4 x = *reinterpret_cast<const float4 *>(Ap + 4 * q);
                areg[4 * q + 0] = x.x; areg[4 * q + 1] = x.y; areg[4 * q + 2] = x.z; areg[4 * q + 3] = x.w;
            }
        }
        for (int i = t; i < NE; i += WG) {
            s_k[i] = gkb[E0 + i].x;
            s_e[i] = (uint8_t)(gu[E0 + i] - u0);
        }
#pragma unroll
        for (int q = 0; q < NB4; ++q) reinterpret_cast<float4 *>(rf_lds)[q * WG + t] = bm[q];
        __syncthreads();
        mfma16_t acc[F::CBW];
#pragma unroll
        for (int cb = 0; cb < F::CBW; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
#pragma unroll
        for (int s = 0; s < F::KH; ++s) {
            const float *Brow = rf_lds + (kh * F::KH + s) * R + ln;
#pragma unroll
            for (int cb = 0; cb < F::CBW; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(areg[s], Brow[32 * (cb0 + cb)], acc[cb], 0, 0, 0);
        }
        __syncthreads();                                                      // the slice has been read by everyone
        // register r of lane (kh, ln) is row 8 (r / 4) + 4 kh + r % 4, column ln of its 32 x 32 block
#pragma unroll
        for (int cb = 0; cb < F::CBW; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                rf_lds[(32 * rb + 8 * (r / 4) + 4 * kh + r % 4) * LDT + 32 * (cb0 + cb) + ln] = acc[cb][r];
        __syncthreads();
        // second product: rows (j1, j2) of T0 (R values each) against G3[i3]
        {
            float4 o[N1];
#pragma unroll
            for (int j = 0; j < N1; ++j) o[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (!F::EARLY_C) {
#pragma unroll
                for (int i = 0; i < F::BQ; ++i) cv[i] = Cp[i * F::NBQ];
            }
#pragma unroll
            for (int i = 0; i < F::BQ; ++i) {
                const float4 c = cv[i];
#pragma unroll
                for (int j = 0; j < N1; ++j) {
                    const float tv = rf_lds[(ee * N1 + j) * LDT + i * F::NBQ + bq];
                    o[j].x = fmaf(tv, c.x, o[j].x); o[j].y = fmaf(tv, c.y, o[j].y);
                    o[j].z = fmaf(tv, c.z, o[j].z); o[j].w = fmaf(tv, c.w, o[j].w);
                }
            }
#pragma unroll
            for (int d = 1; d < F::NBQ; d <<= 1)
#pragma unroll
                for (int j = 0; j < N1; ++j) {
                    o[j].x += __shfl_xor(o[j].x, d); o[j].y += __shfl_xor(o[j].y, d);
                    o[j].z += __shfl_xor(o[j].z, d); o[j].w += __shfl_xor(o[j].w, d);
                }
            if (on) {
#pragma unroll
                for (int j = 0; j < N1; ++j)
                    if (bq == j % F::NBQ)                                     // the threads of a row share out its j1
                        *reinterpret_cast<float4 *>(rows_out + (size_t)(u0 + ee) * C::N + (j * N2 + j2) * 4) = o[j];
            }
        }
        // the kept copies of T0, t0[k][j1][j2][R]: GL threads per position, four positions side by side (a hot row's two
        // thousand positions are all in this workgroup: one at a time they took 80 us)
        // (stored past the caches: most are never read again, and slices and rows stay there instead; 100 positions per bag at rank 64,
        // 210 MB, step 239.0 -> 234.7 us, cached multi-hot, 74 MB, 133.9 -> 131.7)
        {
            constexpr int NG = WG / F::GL, NF = 4;
            const int g = t / F::GL, f = t % F::GL, fj = f / (R / 4), col = 4 * (f % (R / 4));
            for (int i = g; i < NE; i += NF * NG) {
                int k[NF];
                float2 a[NF], b[NF];
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    const int x = min(i + q * NG, NE - 1), at = (s_e[x] * N1 + fj) * LDT + col;
                    k[q] = s_k[x];
                    a[q] = *reinterpret_cast<const float2 *>(rf_lds + at);
                    b[q] = *reinterpret_cast<const float2 *>(rf_lds + at + 2);
                }
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    if (i + q * NG < NE)
                        __builtin_nontemporal_store(rw_f4{a[q].x, a[q].y, b[q].x, b[q].y},
                                                    reinterpret_cast<rw_f4 *>(t0_out + ((size_t)k[q] * N1 + fj) * COLS + j2 * R + col));
            }
        }
        __syncthreads();                                                      // LDS is reused by the next tile
    }
}

// The sum over positions [k0, k1) of alpha[k] rows[inv[k]] by a wave (k0 and k1 the same for all its lanes): it looks at up to 64 positions
// at once, then lane (sub, f) adds float4 f of every (64 / (N/4))-th of them, four in flight; every sub ends with the sum.  With a cache
// (lines), the line ~inv[k] where that is not negative.
__device__ __forceinline__ float4 rw_pool_wave(int N, const float *__restrict__ rows, const int *__restrict__ inv, const float *__restrict__ lines,
                                               const float *__restrict__ alpha, int k0, int k1)
{
    const int lane = threadIdx.x & 63;
    const int nq = N / 4, per = WAVE / nq;                                    // N a power of two <= 256
    const int f = lane % nq, sub = lane / nq;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int kc = k0; kc < k1; kc += WAVE) {
        const int cnt = min(WAVE, k1 - kc), pc = kc + min(lane, cnt - 1);
        const int myu = inv[pc];
        const float myw = alpha ? alpha[pc] : 1.f;
        for (int qb = 0; qb < cnt; qb += 4 * per) {                            // uniform: every lane takes part in the shuffles
            const int q0 = qb + sub;
            float4 x[4];
            float wgt[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int pi = min(q0 + q * per, cnt - 1);
                wgt[q] = __shfl(myw, pi);
                const int u = __shfl(myu, pi);
                x[q] = *reinterpret_cast<const float4 *>((lines && u < 0 ? lines + (size_t)~u * N : rows + (size_t)u * N) + 4 * f);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q0 + q * per < cnt) {
                    acc.x = fmaf(wgt[q], x[q].x, acc.x); acc.y = fmaf(wgt[q], x[q].y, acc.y);
                    acc.z = fmaf(wgt[q], x[q].z, acc.z); acc.w = fmaf(wgt[q], x[q].w, acc.w);
                }
        }
    }
    for (int d = nq; d < WAVE; d <<= 1) {
        acc.x += __shfl_xor(acc.x, d); acc.y += __shfl_xor(acc.y, d);
        acc.z += __shfl_xor(acc.z, d); acc.w += __shfl_xor(acc.w, d);
    }
    return acc;
}

// out[bag] = sum over the bag's positions of alpha[k] rows[inv[k]], one wave per bag
__global__ __launch_bounds__(WG) void rw_pool_kernel(int N, const float *__restrict__ rows, const int *__restrict__ inv, const float *__restrict__ lines,
                                                     const int64_t *__restrict__ offsets, int n_bags, const float *__restrict__ alpha,
                                                     float *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const int bag = blockIdx.x * NWAVE + (threadIdx.x >> 6);
    if (bag >= n_bags) return;                                                // uniform in the wave
    const int k0 = offsets ? (int)offsets[bag] : bag, k1 = offsets ? (int)offsets[bag + 1] : bag + 1;
    const float4 acc = rw_pool_wave(N, rows, inv, lines, alpha, k0, k1);
    if (lane < N / 4) *reinterpret_cast<float4 *>(out + (size_t)bag * N + 4 * lane) = acc;
}

// The same for short bags, fewer than RW_POOL_SHORT positions on average: LANES lanes per bag, so that a wave has several bags and few of
// its lanes idle.  A bag's sums are those of rw_pool_wave, in its order, so that its result does not depend on the other bags: sum s of the
// PER = WAVE / (N / 4) is of positions s, s + PER, ..., and they are added in pairs.  Four times as many sums as lanes have a float4: a lane has
// four of them.  Fewer lanes (PAIRS): a bag has at most one position for every sum, and four of them are added as soon as they are there.
// A bag of more than MOST positions is the whole wave's.
// Neighbouring bags are in different waves: batches come sorted by length, and a wave adds up its long bags one after the other.  A wave per
// bag / neighbours in a wave / this: 16,384 bags sorted by length, Pareto law up to 500, (4,4,4) 66.5 / 126.5 / 65.0 us, 32,768 of (2,2,4)
// 52.4 / 67.4 / 45.5, 16 of 1,000 positions side by side among 98,288 of one 69 / 276 / 52; where no long ones meet 0 to 2 us more than neighbours.
// A forward pass, a wave per bag / this: (4,4,4) rank 32, 16,384 bags of 1-8 39.6 / 37.0 us, of none or 20 38.0 / 38.1, of none or 40 37.4 / 39.5, by a
// Pareto law up to 64 39.0 / 39.8; (2,2,4) rank 32, 32,768 of 1-8 43.1 / 35.3, of none or 20 39.0 / 35.4, 196,608 of one 95 / 41.8 (16 lanes
// 50.6), 65,536 by a Pareto law up to 64 58.4 / 45.9.  Beyond six on average: (4,4,4) 8,192 of 0-20 43.0 / 43.8, rank 64 4,096 64.2 / 65.4; (2,2,4),
// where it is ahead still, 16,384 of 0-20 40.5 / 38.0.
constexpr int RW_POOL_SHORT = 6, RW_POOL_SHORTEST = 2, RW_POOL_LANES = 16, RW_POOL_MOST = 32;
template <int N, int LANES, int MOST>
__global__ __launch_bounds__(WG) void rw_pool_short_kernel(const float *__restrict__ rows, const int *__restrict__ inv, const float *__restrict__ lines,
                                                           const int64_t *__restrict__ offsets, int n_bags, const float *__restrict__ alpha,
                                                           float *__restrict__ out)
{
    constexpr int NQ = N / 4, PER = WAVE / NQ, BAGS = WAVE / LANES, SUBS = LANES / NQ, NA = 4;
    constexpr bool PAIRS = NA * SUBS < PER;
    constexpr int NF = SUBS == 1 && !PAIRS ? 2 * NA : NA;                     // rows in flight
    static_assert(PAIRS ? LANES == NA && PER == 4 * NA && MOST <= PER : NA * SUBS == PER, "the sums of rw_pool_wave");
    const int lane = threadIdx.x & 63, l = lane % LANES, f = lane % NQ, sub = l / NQ;
    const int wave = blockIdx.x * NWAVE + (threadIdx.x >> 6), waves = (int)(((int64_t)n_bags + BAGS - 1) / BAGS);
    if (wave >= waves) return;                                                // uniform in the wave
    const int64_t bag = (int64_t)(lane / LANES) * waves + wave;
    const bool on = bag < n_bags;
    const int k0 = !on ? 0 : offsets ? (int)offsets[bag] : (int)bag, k1 = !on ? 0 : offsets ? (int)offsets[bag + 1] : (int)bag + 1;
    const bool wide = k1 - k0 > MOST;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [](const float4 &x, const float4 &y) { return make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w); };
    float4 acc[NA], half[2] = {zero, zero};
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[q] = zero;
    for (int kc = k0; kc < k1 && !wide; kc += LANES) {                        // (all lanes of a bag go the same way)
        const int cnt = min(LANES, k1 - kc), pc = kc + min(l, cnt - 1);
        const int myu = inv[pc];
        const float myw = alpha ? alpha[pc] : 1.f;
        for (int qb = 0; qb < cnt; qb += NF * SUBS) {
            const int q0 = qb + NF * sub;
            float wgt[NF];
            float4 x[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                const int pi = lane - l + min(q0 + q, cnt - 1), u = __shfl(myu, pi);
                wgt[q] = __shfl(myw, pi);
                x[q] = *reinterpret_cast<const float4 *>((lines && u < 0 ? lines + (size_t)~u * N : rows + (size_t)u * N) + 4 * f);
            }
#pragma unroll
            for (int q = 0; q < NF; ++q)
                if (q0 + q < cnt) {
                    float4 &to = acc[q % NA];
                    to.x = fmaf(wgt[q], x[q].x, to.x); to.y = fmaf(wgt[q], x[q].y, to.y);
                    to.z = fmaf(wgt[q], x[q].z, to.z); to.w = fmaf(wgt[q], x[q].w, to.w);
                }
        }
        if constexpr (PAIRS) {
            const float4 four = add(add(acc[0], acc[1]), add(acc[2], acc[3]));
            if (kc - k0 < PER / 2) half[0] = add(half[0], four);
            else half[1] = add(half[1], four);
#pragma unroll
            for (int q = 0; q < NA; ++q) acc[q] = zero;
        }
    }
    float4 sum = PAIRS ? add(half[0], half[1]) : add(add(acc[0], acc[1]), add(acc[2], acc[3]));
#pragma unroll
    for (int d = NQ; d < LANES; d <<= 1) {
        sum.x += __shfl_xor(sum.x, d); sum.y += __shfl_xor(sum.y, d);
        sum.z += __shfl_xor(sum.z, d); sum.w += __shfl_xor(sum.w, d);
    }
    uint64_t left = __ballot(wide && l == 0);
    while (left) {                                                            // uniform
        const int j = __builtin_ctzll(left);
        left &= left - 1;
        const float4 all = rw_pool_wave(N, rows, inv, lines, alpha, __builtin_amdgcn_readlane(k0, j), __builtin_amdgcn_readlane(k1, j));
        if (lane / LANES == j / LANES) sum = all;
    }
    if (on && sub == 0) *reinterpret_cast<float4 *>(out + (size_t)bag * N + 4 * f) = sum;
}

template <int N>
static inline void rw_pool(const float *rows, const int *inv, const float *lines, const int64_t *off, int n_bags, int64_t L, const float *alpha,
                           float *out, hipStream_t st)
{
    constexpr int LANES = RW_POOL_LANES;
    auto grid = [&](int lanes) { return dim3((unsigned)(((int64_t)n_bags * lanes + WG - 1) / WG)); };
    if constexpr (N / 4 < LANES)
        if (L < (int64_t)RW_POOL_SHORTEST * n_bags) {
            hipLaunchKernelGGL((rw_pool_short_kernel<N, N / 4, WAVE / (N / 4)>), grid(N / 4), dim3(WG), 0, st, rows, inv, lines, off, n_bags, alpha, out);
            return;
        }
    if (L < (int64_t)RW_POOL_SHORT * n_bags)
        hipLaunchKernelGGL((rw_pool_short_kernel<N, LANES, RW_POOL_MOST>), grid(LANES), dim3(WG), 0, st, rows, inv, lines, off, n_bags, alpha, out);
    else
        hipLaunchKernelGGL(rw_pool_kernel, dim3((n_bags + NWAVE - 1) / NWAVE), dim3(WG), 0, st, N, rows, inv, lines, off, n_bags, alpha, out);
}

// ---- backward --------------------------------------------------------------------------------------------------------

// dym[u] = sum over the positions of row u of alpha[k] grad_out[bag(k)].  A workgroup has RM_ROWS values of u; a run of
// positions is cut into pieces of 8 or 16, N / 4 lanes add a piece up, and the pieces of a long run (a hot row) meet in LDS.
constexpr int RM_ROWS = 64;

template <int N, int T>
__global__ __launch_bounds__(T) void rw_merge_kernel(int L, const int4 *__restrict__ rec, const int2 *__restrict__ gkb,
                                                      const float *__restrict__ alpha, const float *__restrict__ grad_out,
                                                      float *__restrict__ dym)
{
    constexpr int NQ = N / 4, NG = T / NQ, RM_PIECE = N > 16 ? 8 : 16, RM_ROOM = 128;
    __shared__ int s_piece[RM_ROWS + 1], s_first[RM_ROWS], s_cnt[RM_ROWS];
    __shared__ __align__(16) float s_part[RM_ROOM * N];
    const int t = threadIdx.x, lane = t & 63, g = t / NQ, f = t % NQ, u0 = blockIdx.x * RM_ROWS;
    if (t < RM_ROWS) {                                                        // the first wave
        const int4 r = rec[min(u0 + t, L - 1)];
        const int cnt = u0 + t < L ? r.w : 0, np = (cnt + RM_PIECE - 1) / RM_PIECE;
        s_first[t] = r.z; s_cnt[t] = cnt;
        int inc = np;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d);
            if (lane >= d) inc += o;
        }
        s_piece[t] = inc - np;
        if (t == RM_ROWS - 1) s_piece[RM_ROWS] = inc;
    }
    __syncthreads();
    const int np = s_piece[RM_ROWS];
    for (int p0 = 0; p0 < np; p0 += RM_ROOM) {                                // uniform
        const int p1 = min(np, p0 + RM_ROOM);
        for (int pc = p0 + g; pc < p1; pc += NG) {
            int lo = 0, hi = RM_ROWS;                                         // last row with s_piece <= pc: it has that piece
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_piece[mid] <= pc) lo = mid; else hi = mid;
            }
            const int c0 = (pc - s_piece[lo]) * RM_PIECE, n = min(RM_PIECE, s_cnt[lo] - c0), b = s_first[lo] + c0;
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
            auto add = [&](auto nf) {
                constexpr int NF = decltype(nf)::value;                        // loads in flight (clamped: none is conditional)
                for (int i = 0; i < n; i += NF) {
                    int2 kb[NF];
                    float4 x[NF];
                    float wt[NF];
#pragma unroll
                    for (int q = 0; q < NF; ++q) kb[q] = gkb[b + min(i + q, n - 1)];
#pragma unroll
                    for (int q = 0; q < NF; ++q) {
                        x[q] = *reinterpret_cast<const float4 *>(grad_out + (size_t)kb[q].y * N + 4 * f);
                        wt[q] = alpha ? alpha[kb[q].x] : 1.f;
                    }
#pragma unroll
                    for (int q = 0; q < NF; ++q)
                        if (i + q < n) {
                            sum.x = fmaf(wt[q], x[q].x, sum.x); sum.y = fmaf(wt[q], x[q].y, sum.y);
                            sum.z = fmaf(wt[q], x[q].z, sum.z); sum.w = fmaf(wt[q], x[q].w, sum.w);
                        }
                }
            };
            if (n <= 2) add(std::integral_constant<int, 2>{});
            else add(std::integral_constant<int, 8>{});
            if (s_cnt[lo] <= RM_PIECE) *reinterpret_cast<float4 *>(dym + (size_t)(u0 + lo) * N + 4 * f) = sum;
            else *reinterpret_cast<float4 *>(s_part + (pc - p0) * N + 4 * f) = sum;
        }
        __syncthreads();
        for (int e = g; e < RM_ROWS; e += NG) {
            if (s_cnt[e] <= RM_PIECE) continue;
            const int b = max(s_piece[e], p0), c = min(s_piece[e + 1], p1);
            if (b >= c) continue;
            float4 *dst = reinterpret_cast<float4 *>(dym + (size_t)(u0 + e) * N + 4 * f);
            float4 sum = b > s_piece[e] ? *dst : make_float4(0.f, 0.f, 0.f, 0.f);
            for (int q = b; q < c; ++q) {
                const float4 x = *reinterpret_cast<const float4 *>(s_part + (q - p0) * N + 4 * f);
                sum.x += x.x; sum.y += x.y; sum.z += x.z; sum.w += x.w;
            }
            *dst = sum;
        }
        __syncthreads();
    }
}

template <typename C, int ROWS_>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(BoCfg<C, ROWS_>::WGS_PER_CU, BoCfg<C, ROWS_>::WGS_PER_CU))) void rw_tile_kernel(
    Params p, const float *__restrict__ G1, const float *__restrict__ G2, const float *__restrict__ G3, int L,
    const float *__restrict__ dym, const int4 *__restrict__ rec, const int4 *__restrict__ tiles, const int *__restrict__ tile_base,
    float *__restrict__ part2, float *__restrict__ pbuf, const float *src2, float *dst2, float mul)
{
    using F = BoCfg<C, ROWS_>;
    constexpr int N1 = C::N1, N2 = C::N2, R = C::R, N = C::N, COLS = C::COLS, TP = F::TP;
    constexpr int LDA = F::LDA, LDT = F::LDT, LDB = F::LDB, NQ = N / 4;
    extern __shared__ __align__(16) float bo_lds[];
    float *dyl = bo_lds;                              // [TP][N]      summed upstream gradients of the rows
    float *As = dyl + F::DY_FLOATS;                   // [128][LDA]   stacked rows of G1
    float *dT = As + F::ROWS * LDA;                   // [128][LDT]   dT0' for the current j2
    float *Bl = dT + F::ROWS * LDT;                   // [R][LDB]     Bm[a][(j2, .)]
    __shared__ int s_ti2[BO_MAX_CHUNK], s_tlo[BO_MAX_CHUNK], s_tn[BO_MAX_CHUNK];   // the workgroup's tiles: slice, first item, items
    __shared__ int s_i1[2][TP], s_i3[2][TP];          // digits of the rows of this tile and of the next one
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int ln = lane & 31, kh = lane >> 5;
    const int blk = w % F::NB, ks = w / F::NB;        // this wave adds rows [ks ROWS / KS, (ks + 1) ROWS / KS) into block blk
    const int ab1 = blk / F::RB, bb1 = blk % F::RB;
    const int rb = w % F::RBK, ab0 = (w / F::RBK) * F::ABW;   // this wave's block of P: rows 32 rb .., column blocks ab0 .. ab0 + ABW - 1

    const int used = tile_base[p.m2];
    const int ch = bo_chunk(used, gridDim.x);
    const int tbeg = blockIdx.x * ch, tend = min(used, tbeg + min(ch, BO_MAX_CHUNK));
    if (tbeg >= tend) return;                         // uniform
    if (t < tend - tbeg) {
        const int4 td = tiles[tbeg + t];
        // (guards against a table that no pre-pass wrote: such a tile ends the workgroup's work)
        const bool ok = td.z > 0 && (unsigned)td.x < (unsigned)p.m2 && td.y >= 0 && td.z <= TP && td.y + td.z <= L;
        s_ti2[t] = ok ? td.x : -1; s_tlo[t] = ok ? td.y : 0; s_tn[t] = ok ? td.z : 0;
    }
    bo_lds_barrier();

    // ---- the pipeline's registers: records of the tile after next, operands of the next tile ----
    // (plain floats and ints: arrays of vector types that lambdas take by reference end up in scratch memory)
    int pin_i1 = 0, pin_i3 = 0;
    float nxt_dy[F::NDY][4], nxt_a[F::NA4][4], nxt_cv[F::BQ][4], cv[F::BQ][4];
    constexpr int NB4 = R * R / 4 / WG;
    float bm[NB4][4];
    auto ld4 = [](const float *src, float (&d)[4]) __attribute__((always_inline)) {
        const float4 v = *reinterpret_cast<const float4 *>(src);
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    };
    const int ee = t / F::NBQ, bq = t % F::NBQ;        // thread (position ee, bq) of the dT0' product: rows b = NBQ i + bq of G3[i3]

    auto load_records = [&](int lo) __attribute__((always_inline)) {
        if (t < TP) {
            const int4 pi = rec[min(lo + t, L - 1)];
            pin_i1 = pi.x; pin_i3 = pi.y;
        }
    };
    auto publish_records = [&](int n, int set) __attribute__((always_inline)) {
        if (t < TP) {
            const bool on = t < n;
            s_i1[set][t] = on ? min(max(pin_i1, 0), p.m1 - 1) : 0;
            s_i3[set][t] = on ? min(max(pin_i3, 0), p.m3 - 1) : 0;
        }
    };
    auto fetch_bm = [&](int i2, int j2) __attribute__((always_inline)) {
        const float *src = G2 + (size_t)i2 * C::sB + j2 * R;
#pragma unroll
        for (int q = 0; q < NB4; ++q) {
            const int i = q * WG + t, a = i / (R / 4), b4 = 4 * (i % (R / 4));
            ld4(src + a * COLS + b4, bm[q]);
        }
    };
    auto issue_operands = [&](int set, int lo) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < F::NDY; ++q) {
            const int i = q * WG + t, e = i / NQ, f = i % NQ;
            ld4(dym + (size_t)min(lo + e, L - 1) * N + 4 * f, nxt_dy[q]);
        }
#pragma unroll
        for (int q = 0; q < F::NA4; ++q) {
            const int i = q * WG + t, row = i / (R / 4), a4 = 4 * (i % (R / 4)), e = row / N1, j1 = row % N1;
            ld4(G1 + (size_t)s_i1[set][e] * C::sA + j1 * R + a4, nxt_a[q]);
        }
        const float *Cp = G3 + (size_t)s_i3[set][ee] * C::sC + 4 * bq;
#pragma unroll
        for (int i = 0; i < F::BQ; ++i) ld4(Cp + 4 * i * F::NBQ, nxt_cv[i]);
    };
    // the operands of a tile of n positions to LDS and to cv[] (positions past the end: zeros)
    auto commit_operands = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < F::NDY; ++q) {
            const int i = q * WG + t, e = i / NQ, f = i % NQ;
            *reinterpret_cast<float4 *>(dyl + e * N + 4 * f) =                // (selected per component: a select of float4s goes through memory)
                make_float4(e < n ? nxt_dy[q][0] : 0.f, e < n ? nxt_dy[q][1] : 0.f, e < n ? nxt_dy[q][2] : 0.f, e < n ? nxt_dy[q][3] : 0.f);
        }
#pragma unroll
        for (int q = 0; q < F::NA4; ++q) {
            const int i = q * WG + t, row = i / (R / 4), a4 = 4 * (i % (R / 4)), e = row / N1;
            const bool on = e < n;
            *reinterpret_cast<float4 *>(As + row * LDA + a4) =
                make_float4(on ? nxt_a[q][0] : 0.f, on ? nxt_a[q][1] : 0.f, on ? nxt_a[q][2] : 0.f, on ? nxt_a[q][3] : 0.f);
        }
#pragma unroll
        for (int i = 0; i < F::BQ; ++i)
#pragma unroll
            for (int x = 0; x < 4; ++x) cv[i][x] = ee < n ? nxt_cv[i][x] : 0.f;
    };

    mfma16_t acc1[N2];
    int cur = -1;
    auto flush1 = [&]() __attribute__((always_inline)) {                       // (uniform)
        if (cur < 0) return;
        // a slice whose tiles are all this workgroup's is finished here; else the stretch leaves a part, under a new number for
        // every stretch (the slice or the workgroup has moved on)
        const bool whole = tile_base[cur] >= tbeg && tile_base[cur + 1] <= tend;
        const float *old = src2 + (size_t)cur * C::sB;
        float *out = whole ? dst2 + (size_t)cur * C::sB : part2 + (size_t)(cur + (int)blockIdx.x) * C::sB;
        if constexpr (F::KS == 1) {
#pragma unroll
            for (int j2 = 0; j2 < N2; ++j2) {
                const size_t at = (size_t)(32 * ab1 + 4 * kh) * COLS + j2 * R + 32 * bb1 + ln;
                float x[16];
                if (whole) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[r] = old[at + (size_t)(8 * (r / 4) + r % 4) * COLS];
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) out[at + (size_t)(8 * (r / 4) + r % 4) * COLS] = whole ? fmaf(mul, acc1[j2][r], x[r]) : acc1[j2][r];
            }
        } else {
            // the waves' partial blocks through the dT0' area (free between tiles): element (row, col) of wave w's block is
            // value r = 4 (row / 8) + row % 4 of lane 32 ((row / 4) % 2) + col; thread (row, four columns) adds the KS partials
            // of a block in wave order and stores a float4
#pragma unroll
            for (int j2 = 0; j2 < N2; ++j2) {
#pragma unroll
                for (int r = 0; r < 16; ++r) dT[w * 1024 + r * 64 + lane] = acc1[j2][r];
                bo_lds_barrier();
                for (int x = t; x < F::NB * 256; x += WG) {
                    const int b = x / 256, row = (x % 256) / 8, c4 = 4 * (x % 8);
                    const int at = (4 * (row / 8) + row % 4) * 64 + 32 * ((row / 4) % 2) + c4;
                    float4 sum = *reinterpret_cast<const float4 *>(&dT[b * 1024 + at]);
#pragma unroll
                    for (int q = 1; q < F::KS; ++q) {
                        const float4 v = *reinterpret_cast<const float4 *>(&dT[(b + F::NB * q) * 1024 + at]);
                        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
                    }
                    const size_t to = (size_t)(32 * (b / F::RB) + row) * COLS + j2 * R + 32 * (b % F::RB) + c4;
                    if (whole) {
                        const float4 o = *reinterpret_cast<const float4 *>(old + to);
                        sum = make_float4(fmaf(mul, sum.x, o.x), fmaf(mul, sum.y, o.y), fmaf(mul, sum.z, o.z), fmaf(mul, sum.w, o.w));
                    }
                    *reinterpret_cast<float4 *>(out + to) = sum;
                }
                bo_lds_barrier();
            }
        }
    };

    // ---- prologue: the first tile's operands, the second tile's records ----
    {
        load_records(s_tlo[0]);
        publish_records(s_tn[0], 0);
        bo_lds_barrier();
        issue_operands(0, s_tlo[0]);
        if (s_ti2[0] >= 0) fetch_bm(s_ti2[0], 0);
        if (tbeg + 1 < tend) load_records(s_tlo[1]);
        commit_operands(s_tn[0]);
        bo_lds_barrier();
    }
    int sc = 0;
    for (int tile = tbeg; tile < tend; ++tile, sc ^= 1) {
        const int i2 = s_ti2[tile - tbeg], n = s_tn[tile - tbeg], lo0 = s_tlo[tile - tbeg];
        if (i2 < 0) break;                                                 // uniform
        const bool has_next = tile + 1 < tend;
        const int i2n = has_next ? s_ti2[tile + 1 - tbeg] : -1, nn = has_next ? s_tn[tile + 1 - tbeg] : 0;
        if (i2 != cur) {
            flush1();
            cur = i2;
#pragma unroll
            for (int j2 = 0; j2 < N2; ++j2)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc1[j2][r] = 0.f;
        }
        // the next tile: its records to LDS, its operands on their way, the records of the one after it too
        if (has_next) {
            publish_records(nn, sc ^ 1);
            bo_lds_barrier();
            issue_operands(sc ^ 1, s_tlo[tile + 1 - tbeg]);
            if (tile + 2 < tend) load_records(s_tlo[tile + 2 - tbeg]);
        }

        mfma16_t accp[F::ABW];                                             // P: rows 32 rb .. 32 rb + 31, this wave's column blocks
#pragma unroll
        for (int ab = 0; ab < F::ABW; ++ab)
#pragma unroll
            for (int r = 0; r < 16; ++r) accp[ab][r] = 0.f;

#pragma unroll
        for (int j2 = 0; j2 < N2; ++j2) {
            // Bm[a][(j2, b)] to LDS (it came through registers: the part for the next j2, or for the next tile, is fetched
            // while the products of this one run)
#pragma unroll
            for (int q = 0; q < NB4; ++q) {
                const int i = q * WG + t, a = i / (R / 4), b4 = 4 * (i % (R / 4));
                *reinterpret_cast<float4 *>(Bl + a * LDB + b4) = make_float4(bm[q][0], bm[q][1], bm[q][2], bm[q][3]);
            }
            if (j2 + 1 < N2) fetch_bm(i2, j2 + 1);
            else if (i2n >= 0) fetch_bm(i2n, 0);
            // dT0'[(ee, j1)][b] for this j2
#pragma unroll
            for (int j1 = 0; j1 < N1; ++j1) {
                const float4 dy = *reinterpret_cast<const float4 *>(dyl + ee * N + (j1 * N2 + j2) * 4);
#pragma unroll
                for (int i = 0; i < F::BQ; ++i) {
                    dT[(ee * N1 + j1) * LDT + i * F::NBQ + bq] = fmaf(dy.x, cv[i][0], fmaf(dy.y, cv[i][1], fmaf(dy.z, cv[i][2], dy.w * cv[i][3])));
                }
            }
            bo_lds_barrier();
            // the part of dG2: block blk of the R x R result for this j2, over this wave's share of the stacked rows (stopping at
            // the tile's last row, a quarter of the share at a time, was measured: slower, the loop's loads no longer run ahead)
            {
                constexpr int RW = F::ROWS / F::KS;
#pragma unroll
                for (int s = 0; s < RW / 2; ++s) {
                    const int row = ks * RW + kh * (RW / 2) + s;
                    acc1[j2] = __builtin_amdgcn_mfma_f32_32x32x2f32(As[row * LDA + 32 * ab1 + ln], dT[row * LDT + 32 * bb1 + ln],
                                                                   acc1[j2], 0, 0, 0);
                }
            }
            // P += dT0' Bm^T over the columns of this j2
#pragma unroll
            for (int s = 0; s < R / 2; s += 4) {
                const float2 av0 = *reinterpret_cast<const float2 *>(&dT[(32 * rb + ln) * LDT + kh * (R / 2) + s]);
                const float2 av1 = *reinterpret_cast<const float2 *>(&dT[(32 * rb + ln) * LDT + kh * (R / 2) + s + 2]);
#pragma unroll
                for (int ab = 0; ab < F::ABW; ++ab) {
                    const float4 bv = *reinterpret_cast<const float4 *>(&Bl[(32 * (ab0 + ab) + ln) * LDB + kh * (R / 2) + s]);
                    accp[ab] = __builtin_amdgcn_mfma_f32_32x32x2f32(av0.x, bv.x, accp[ab], 0, 0, 0);
                    accp[ab] = __builtin_amdgcn_mfma_f32_32x32x2f32(av0.y, bv.y, accp[ab], 0, 0, 0);
                    accp[ab] = __builtin_amdgcn_mfma_f32_32x32x2f32(av1.x, bv.z, accp[ab], 0, 0, 0);
                    accp[ab] = __builtin_amdgcn_mfma_f32_32x32x2f32(av1.y, bv.w, accp[ab], 0, 0, 0);
                }
            }
            bo_lds_barrier();                                               // dT0' and Bm are rewritten for the next j2
        }
        // the G1 gradients of the rows: pbuf[u][j1][a]
#pragma unroll
        for (int ab = 0; ab < F::ABW; ++ab)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 32 * rb + 8 * (r / 4) + 4 * kh + r % 4, e = row / N1, j1 = row % N1;
                if (e < n) pbuf[((size_t)(lo0 + e) * N1 + j1) * R + 32 * (ab0 + ab) + ln] = accp[ab][r];
            }
        if (has_next) commit_operands(nn);
        bo_lds_barrier();                                                   // the next tile's operands are in place; this tile's records are free
    }
    flush1();
}

// ---- the sums that finish the three cores -----------------------------------------------------------------------------
// Workgroups [0, cwgs): gradients of cached rows; then, counted from there, [0, m1 + m3): the first piece (rw_piece rows) of a slice of the third core, which take longest, or of the first; the next `extra`: what slices
// have beyond that; the rest: the parts of the slices of the second core.  A slice of one piece (nearly all, where rows repeat:
// equal rows are one) is finished on the spot; of a longer one every piece leaves a partial sum and the workgroup that arrives
// last adds them, in their order.  How many extra pieces there are is only known on the device: as many workgroups are started
// for them as there can be, or as the device runs at once (with 64 of them a step of 300,000 uniform
// positions, Kaggle-shaped at rank 32, took 901 us, 600 of them here; so it takes 290).
constexpr int RS_MAX_EXTRA = 1024;
// Windows of a cached row that its lanes add up alone: 16 rounds of loads.  A hot row's of a long stream would be hundreds.  (4,4,4) at
// rank 32, step, slices' lists / alone / shared: the only cached row with 90 % of 300,000 positions 200 / 201 / 178 us, of 1,000,000
// 549 / 608 / 520; one of 1,000 with 80 % 220 / 210 / 200 and 585 / 589 / 527, of 8,000 204 / 190 / 183 and 541 / 560 / 511; no hot row: as it
// was (300,000 positions, 8,000 rows, 233 / 232).  Shorter streams do without, and without its code: with it, whether it
// runs or not, 163,840 positions take 131 us instead of 130.
constexpr int RW_ALONE = 128;
constexpr int64_t RW_SHARE_MIN_L = 262144;

struct RsArgs {
    const float *src[3];
    float *dst[3];
    float mul;
    int nwg;                 // workgroups of the tile kernel
    int piece, extra;        // rows of a piece (RW_PIECE at most); workgroups for the extra pieces
    int K, cwgs;             // cached rows, and the workgroups that add their gradients up
    float *lines;            // lines[slot] += mul * gradient
};

// CACHED: there is a cache; SHARE: lanes share the windows of its hot rows.
template <typename C, bool CACHED, bool SHARE>
__global__ __launch_bounds__(RW_T) __attribute__((amdgpu_waves_per_eu(4))) void rw_sum_kernel(Params p, RowsWs ws, RsArgs a, const float *__restrict__ t0, const float *__restrict__ dym,
                                                      const float *__restrict__ pbuf, const int2 *__restrict__ l13)
{
    constexpr int N = C::N, R = C::R, NJ = C::N1 * C::N2, sA4 = C::sA / 4, sB4 = C::sB / 4;
    constexpr int WMAX = C::sA > C::sC ? C::sA : C::sC;
    static_assert(N <= WAVE, "a lane per value of a row");
    static_assert(RW_PIECE == RW_T, "a list entry per thread");
    __shared__ __align__(16) float s_red[RW_T * 4];
    __shared__ int2 s_list[RW_PIECE];
    __shared__ __align__(16) float s_dy[RW_NW][4 * N];
    __shared__ int s_tmp[RW_NW], s_at[3], s_last;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), m13 = p.m1 + p.m3;

    if (CACHED && (int)blockIdx.x < a.cwgs) {
        // The gradient of a cached row: over the windows of its bin, in their order; N / 4 lanes per slot, eight windows in flight.
        // In a long stream what has more than RW_ALONE windows is then shared out among all lanes of the workgroup.
        constexpr int NQ = N / 4, NF = 8, GROUPS = RW_T / NQ;
        const int f = t % NQ, g = t / NQ, slot = (int)blockIdx.x * GROUPS + g;
        auto add_up = [&](int j, int w0, int w1, float4 &sum) __attribute__((always_inline)) {
            bool any = false;
            for (int x = w0; x < w1; x += NF) {
                int u[NF];
                float4 v[NF];
#pragma unroll
                for (int q = 0; q < NF; ++q) u[q] = ws.cu[(size_t)min(x + q, w1 - 1) * ws.spb + j];
#pragma unroll
                for (int q = 0; q < NF; ++q) v[q] = *reinterpret_cast<const float4 *>(dym + (size_t)max(u[q], 0) * N + 4 * f);
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    if (x + q < w1 && u[q] >= 0) {
                        sum.x += v[q].x; sum.y += v[q].y; sum.z += v[q].z; sum.w += v[q].w;
                        any = true;
                    }
            }
            return any;
        };
        auto update = [&](int slot, const float4 &sum) __attribute__((always_inline)) {
            const size_t at = (size_t)slot * N + 4 * f;
            const float4 o = *reinterpret_cast<const float4 *>(a.lines + at);
            *reinterpret_cast<float4 *>(a.lines + at) = make_float4(fmaf(a.mul, sum.x, o.x), fmaf(a.mul, sum.y, o.y), fmaf(a.mul, sum.z, o.z), fmaf(a.mul, sum.w, o.w));
        };
        if constexpr (SHARE) {
            if (t == 0) s_last = 0;
            __syncthreads();
        }
        if (slot < a.K) {
            const int w0 = ws.cwin[slot % RW_CBINS], w1 = ws.cwin[slot % RW_CBINS + 1];
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
            if (SHARE && w1 - w0 > RW_ALONE) {
                if (f == 0) s_list[atomicAdd(&s_last, 1)].x = slot;
            } else if (add_up(slot / RW_CBINS, w0, w1, sum)) {
                update(slot, sum);
            }
        }
        if constexpr (!SHARE) return;
        __syncthreads();
        for (int q = 0, n = s_last; q < n; ++q) {                  // uniform
            const int long_slot = s_list[q].x, bin = long_slot % RW_CBINS;
            const int w0 = ws.cwin[bin], nw = ws.cwin[bin + 1] - w0, share = (nw + GROUPS - 1) / GROUPS;
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
            bool any = add_up(long_slot / RW_CBINS, w0 + min(nw, g * share), w0 + min(nw, (g + 1) * share), sum);
            reinterpret_cast<float4 *>(s_red)[t] = sum;
            s_list[t].y = any;
            __syncthreads();
            if (g == 0) {
                for (int x = t + NQ; x < RW_T; x += NQ) {
                    const float4 v = reinterpret_cast<float4 *>(s_red)[x];
                    sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
                    any |= s_list[x].y != 0;
                }
                if (any) update(long_slot, sum);
            }
            __syncthreads();                                       // (s_red is written again)
        }
        return;
    }
    const int wg = (int)blockIdx.x - (CACHED ? a.cwgs : 0);
    if (wg >= m13 + a.extra) {
        // dst[i2] = src[i2] + mul * (parts of slice i2, in the order of their workgroups)
        constexpr int FIN = 2 * RW_T, PER = (sB4 + FIN - 1) / FIN, NP = 8;
        const int vb = wg - m13 - a.extra, i2 = vb / PER, e0 = (vb % PER) * FIN + t;
        if (i2 >= p.m2) return;
        const int tb = ws.tile_base[i2], te = ws.tile_base[i2 + 1], ch = bo_chunk(ws.tile_base[p.m2], a.nwg);
        const float4 *src = reinterpret_cast<const float4 *>(a.src[1]) + (size_t)i2 * sB4;
        float4 *dst = reinterpret_cast<float4 *>(a.dst[1]) + (size_t)i2 * sB4;
        const int b0 = tb / ch, nb = te > tb ? (te - 1) / ch - b0 + 1 : 0;
        if (nb == 1 || (nb == 0 && dst == src)) return;                       // (of one workgroup: the tile kernel has finished it)
        const float4 *part = reinterpret_cast<const float4 *>(ws.part2) + (size_t)(i2 + b0) * sB4;
        int e[2];
        float4 old[2], sum[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            e[f] = min(e0 + f * RW_T, sB4 - 1);
            old[f] = src[e[f]];
            sum[f] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int j = 0; j < nb; j += NP) {                                    // uniform
            float4 x[2][NP];
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int f = 0; f < 2; ++f)
                    x[f][q] = part[(size_t)min(j + q, nb - 1) * sB4 + e[f]];
#pragma unroll
            for (int q = 0; q < NP; ++q)
                if (j + q < nb) {
#pragma unroll
                    for (int f = 0; f < 2; ++f) { sum[f].x += x[f][q].x; sum[f].y += x[f][q].y; sum[f].z += x[f][q].z; sum[f].w += x[f][q].w; }
                }
        }
#pragma unroll
        for (int f = 0; f < 2; ++f)
            if (e0 + f * RW_T < sB4)
                dst[e[f]] = make_float4(fmaf(a.mul, sum[f].x, old[f].x), fmaf(a.mul, sum[f].y, old[f].y), fmaf(a.mul, sum[f].z, old[f].z),
                                        fmaf(a.mul, sum[f].w, old[f].w));
        return;
    }

    // extra piece x of all slices: its slice, and the number of the slice's first extra piece, in s_at (uniform); or, with
    // want_bin >= 0, the latter for that slice
    auto find_extra = [&](int x, int want_bin) {
        constexpr int PB = RW_MAX_M13 / RW_T;
        int v[PB], sum = 0;
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int bin = t * PB + q;
            const int len = bin < m13 ? ws.off13[bin + 1] - ws.off13[bin] : 0;
            v[q] = len > a.piece ? (len - 1) / a.piece : 0;
            sum += v[q];
        }
        int total;
        int at = rw_scan(sum, s_tmp, &total);
        if (t == 0) s_at[2] = total;
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int bin = t * PB + q;
            if (want_bin >= 0 ? bin == want_bin : (x >= at && x < at + v[q])) { s_at[0] = bin; s_at[1] = at; }
            at += v[q];
        }
        __syncthreads();
    };

    // adds rows [i0, i1) of slice `bin` up; the sum's float4 f is in thread f < (row's float4) afterwards
    auto add_up = [&](int bin, int i0, int i1) {
        float4 tot = make_float4(0.f, 0.f, 0.f, 0.f);
        const int n = i1 - i0;
        if (t < n) s_list[t] = l13[i0 + t];                                   // n <= RW_PIECE = RW_T
        __syncthreads();
        if (bin < p.m1) {
            constexpr int NG = RW_T / sA4, NF = 8;
            const int g = t / sA4, f = t % sA4;
            const float4 *pb = reinterpret_cast<const float4 *>(pbuf) + f;
            for (int i = g; i < n; i += NF * NG) {
                float4 x[NF];
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    x[q] = pb[(size_t)s_list[min(i + q * NG, n - 1)].x * sA4];
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    if (i + q * NG < n) { tot.x += x[q].x; tot.y += x[q].y; tot.z += x[q].z; tot.w += x[q].w; }
            }
            reinterpret_cast<float4 *>(s_red)[t] = tot;
            __syncthreads();
            if (t < sA4) {
                for (int q = 1; q < NG; ++q) {
                    const float4 x = reinterpret_cast<float4 *>(s_red)[q * sA4 + t];
                    tot.x += x.x; tot.y += x.y; tot.z += x.z; tot.w += x.w;
                }
            }
        } else {
            // lane (h, b): rows jj = h NJ / H .. of T0 at column b against the upstream gradient, which the wave fetches together with them
            // and reads back from LDS, the same 16 bytes for all lanes of an h; the wave takes every RW_NW-th row of the slice.  (By scalar
            // loads, which come one row at a time when T0 is there, and whose two halves every lane chose between: 164 registers, one workgroup
            // per compute unit, 29 us of this kernel for 8,192 bags of 20 with a cache at (4,4,4) rank 32; so 96, two, 19.  20,000 positions, (2,2,4)
            // rank 32, 6.7 / 5.1; 204,800 at rank 64 30 / 28.  (4,4,4) rank 64 without a cache 88 registers and 118 so, two workgroups either way:
            // held to 93 a step of 8,192 positions takes 85.3 instead of 87.5 us, of 6,500 81.7 instead of 80.4, of 12,000 102.8 instead of 102.2.)
            constexpr int H = WAVE / R > 0 ? WAVE / R : 1, NJH = NJ / H, NF = NJH > 8 ? 2 : 4;
            const int h = H > 1 ? lane / R : 0, b = lane % R;
            float *dyl = s_dy[w];
            for (int i = w; i < n; i += NF * RW_NW) {
                float tv[NF][NJH];
                float dv[NF];
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    const int2 e = s_list[min(i + q * RW_NW, n - 1)];
                    const int uu = __builtin_amdgcn_readfirstlane(e.x);
                    dv[q] = dym[(size_t)uu * N + min(lane, N - 1)];
                    const float *T = t0 + (size_t)__builtin_amdgcn_readfirstlane(e.y) * (NJ * R) + h * NJH * R + b;
#pragma unroll
                    for (int j = 0; j < NJH; ++j) tv[q][j] = T[j * R];
                }
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    if (lane < N) dyl[q * N + lane] = dv[q];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");        // (LDS of one wave is in order: only the compiler has to keep it)
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    if (i + q * RW_NW < n) {                                  // uniform in the wave
#pragma unroll
                    for (int j = 0; j < NJH; ++j) {
                        const float4 d = *reinterpret_cast<const float4 *>(dyl + q * N + 4 * (h * NJH + j));
                        tot.x = fmaf(tv[q][j], d.x, tot.x); tot.y = fmaf(tv[q][j], d.y, tot.y);
                        tot.z = fmaf(tv[q][j], d.z, tot.z); tot.w = fmaf(tv[q][j], d.w, tot.w);
                    }
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                __builtin_amdgcn_wave_barrier();                              // the next rows take their place
            }
            if (H > 1) {
                tot.x += __shfl_xor(tot.x, R); tot.y += __shfl_xor(tot.y, R); tot.z += __shfl_xor(tot.z, R); tot.w += __shfl_xor(tot.w, R);
            }
            reinterpret_cast<float4 *>(s_red)[t] = tot;
            __syncthreads();
            if (t < R)
                for (int q = 1; q < RW_NW; ++q) {
                    const float4 x = reinterpret_cast<float4 *>(s_red)[q * WAVE + t];
                    tot.x += x.x; tot.y += x.y; tot.z += x.z; tot.w += x.w;
                }
        }
        return tot;
    };
    auto finish = [&](int bin, float4 sum, bool none) {
        const bool third = bin >= p.m1;
        const int w4 = third ? R : sA4;
        const size_t at = (size_t)(third ? bin - p.m1 : bin) * w4 + t;
        const float4 *src = reinterpret_cast<const float4 *>(third ? a.src[2] : a.src[0]);
        float4 *dst = reinterpret_cast<float4 *>(third ? a.dst[2] : a.dst[0]);
        if (t >= w4 || (none && dst == src)) return;
        const float4 o = src[at];
        dst[at] = none ? o : make_float4(fmaf(a.mul, sum.x, o.x), fmaf(a.mul, sum.y, o.y), fmaf(a.mul, sum.z, o.z), fmaf(a.mul, sum.w, o.w));
    };
    // a partial sum in place `slot`; whoever arrives last adds all of the slice's up (extra: its first extra piece, -1: unknown)
    auto leave = [&](int bin, float4 sum, int slot, int extra) {
        const bool third = bin >= p.m1;
        const int w4 = third ? R : sA4, len = ws.off13[bin + 1] - ws.off13[bin], np = (len + a.piece - 1) / a.piece;
        if (t < w4) {
            float *to = ws.part13 + (size_t)slot * WMAX + 4 * t;
            __hip_atomic_store(to + 0, sum.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(to + 1, sum.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(to + 2, sum.z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(to + 3, sum.w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // The sum has to be where the whole device meets before this workgroup counts itself as arrived; a barrier alone does not
        // wait for that.  (The stores and the loads below go there by themselves, so no fence has to write the caches back.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (t == 0) {
            s_last = atomicAdd(&ws.arrived[bin], 1u) == (uint32_t)(np - 1);
            if (s_last) atomicExch(&ws.arrived[bin], 0u);                     // (as the pre-pass left it)
        }
        __syncthreads();
        if (!s_last) return;                                                  // uniform
        if (extra < 0) {
            find_extra(0, bin);
            extra = s_at[1];
        }
        float4 tot = make_float4(0.f, 0.f, 0.f, 0.f);
        if (t < w4)
            for (int q = 0; q < np; ++q) {
                const float *src = ws.part13 + (size_t)(q == 0 ? bin : m13 + extra + q - 1) * WMAX + 4 * t;
                tot.x += __hip_atomic_load(src + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                tot.y += __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                tot.z += __hip_atomic_load(src + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                tot.w += __hip_atomic_load(src + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        finish(bin, tot, false);
    };

    if (wg < m13) {
        const int bin = wg < p.m3 ? p.m1 + wg : wg - p.m3, i0 = ws.off13[bin], i1 = ws.off13[bin + 1];
        const float4 sum = add_up(bin, i0, min(i1, i0 + a.piece));
        if (i1 - i0 <= a.piece) finish(bin, sum, i1 == i0);
        else leave(bin, sum, bin, -1);
        return;
    }
    for (int x = wg - m13;; x += a.extra) {
        __syncthreads();
        find_extra(x, -1);
        if (x >= s_at[2]) return;                                             // uniform
        const int bin = s_at[0], first = s_at[1];
        const int i0 = ws.off13[bin] + (x - first + 1) * a.piece;
        __syncthreads();
        const float4 sum = add_up(bin, i0, min(ws.off13[bin + 1], i0 + a.piece));
        leave(bin, sum, m13 + x, first);
    }
}

// ---- host side -------------------------------------------------------------------------------------------------------

// distinct rows per tile: 128 stacked rows
static inline int rw_tp(const Params &p) { return 128 / p.n1; }

// workgroups of the tile kernel: what the compute units hold, and where one would get more tiles than it has room for as often that as
// it takes (524 for the 512 that run at once, as 1,000,000 positions with a cache had it, and the kernel takes twice as long: step at
// (4,4,4) rank 32, hardly a row repeated or cached, 2,800 us, with 1,024 2,460; (2,2,4) rank 64 2,233 / 1,757)
// As many whether a pre-pass runs beside it or not: one call and the two calls of a step have the same sums.  Three for two units below
// 262,144 positions at rank 32, which leave registers for the next batch's pre-pass, against two for one: in two calls on two streams
// 2,048 bags of 100, (2,2,4), 112.7 / 116.1 us, 8,192 of 20, (4,4,4), with a cache 117.5 / 121.6 (on new batches 143.6 / 137.0), without
// 211.5 / 204.9, 10,000 of 20 uniform rows 522 / 470; on one stream 134.2 / 128.4, 144.1 / 135.0, 234.0 / 226.5; in one call 163.3 / 157.6,
// 166.3 / 156.4, 336 / 326; 60,000 positions, (4,4,4), 113.4 / 115.9, 134.9 / 126.0, 168.8 / 159.8.
static inline int rw_tile_wgs(const Params &p, int64_t L, int64_t K)
{
    const int n = (p.R1 >= 64 ? 1 : 2) * bo_compute_units();
    const int least = (rw_tiles(p, L, K, rw_tp(p)) + BO_MAX_CHUNK - 1) / BO_MAX_CHUNK;
    return n > least ? n : (least + n - 1) / n * n;
}

template <typename C, int ROWS_>
static inline hipError_t launch_rw_fwd(const Params &p, const float *G1, const float *G2, const float *G3, int64_t L, const int64_t *off, int n_bags,
                                       const float *alpha, const CacheDev &cache, float *out, float *t0, const RowsWs &ws, hipStream_t st)
{
    const size_t lds = (size_t)RfCfg<C, ROWS_>::LDS_FLOATS * sizeof(float);
    static OncePerDevice once;
    hipError_t e = allow_dynamic_lds(once, (const void *)rw_fwd_kernel<C, ROWS_>, lds);
    if (e != hipSuccess) return e;
    // how many tiles are in use is only known on the device: some workgroups find none, or more than one
    const int tiles = rw_tiles(p, L, cache.K, ROWS_ / C::N1), started = tiles < 2048 ? tiles : 2048;
    hipLaunchKernelGGL((rw_fwd_kernel<C, ROWS_>), dim3(started * C::N2), dim3(WG), lds, st, p, G1, G2, G3, (int)L, ws.rec, ws.gkb, ws.gu,
                       ws.tiles, ws.tile_base, ws.rows, t0);
    rw_pool<C::N>(ws.rows, ws.inv, cache.K ? cache.rows : (const float *)nullptr, off, n_bags, L, alpha, out, st);
    return hipGetLastError();
}

static inline hipError_t rw_fwd(const Params &p, const float *G1, const float *G2, const float *G3, int64_t L, const int64_t *off, int n_bags,
                                const float *alpha, const CacheDev &cache, float *out, float *t0, const RowsWs &ws, hipStream_t st)
{
    switch (fast_config(p)) {
    case 2: return launch_rw_fwd<Cfg224R32, 128>(p, G1, G2, G3, L, off, n_bags, alpha, cache, out, t0, ws, st);
    case 3: return launch_rw_fwd<Cfg224R64, 128>(p, G1, G2, G3, L, off, n_bags, alpha, cache, out, t0, ws, st);
    case 4: return launch_rw_fwd<Cfg444R32, 128>(p, G1, G2, G3, L, off, n_bags, alpha, cache, out, t0, ws, st);
    case 5: return launch_rw_fwd<Cfg444R64, 128>(p, G1, G2, G3, L, off, n_bags, alpha, cache, out, t0, ws, st);
    default: return hipErrorInvalidValue;
    }
}

template <typename C, int ROWS_>
static inline hipError_t launch_rw_bwd(const Params &p, const float *G1, const float *G2, const float *G3, int64_t L, const float *alpha,
                                       const float *go, const float *t0, const float *const src[3], float *const dst[3], float mul, int K, float *lines, const RowsWs &ws,
                                       hipStream_t st)
{
    const size_t lds = bo_lds_bytes<C, ROWS_>();
    static OncePerDevice once;
    hipError_t e = allow_dynamic_lds(once, (const void *)rw_tile_kernel<C, ROWS_>, lds);
    if (e != hipSuccess) return e;
    const int nwg = rw_tile_wgs(p, L, K), cwgs = (int)(((int64_t)K * (C::N / 4) + RW_T - 1) / RW_T), per = (C::sB / 4 + 2 * RW_T - 1) / (2 * RW_T);
    constexpr int MT = C::N > 16 ? 512 : 256;
    hipLaunchKernelGGL((rw_merge_kernel<C::N, MT>), dim3((unsigned)((L + RM_ROWS - 1) / RM_ROWS)), dim3(MT), 0, st, (int)L, ws.rec, ws.gkb, alpha, go,
                       ws.dym);
    hipLaunchKernelGGL((rw_tile_kernel<C, ROWS_>), dim3(nwg), dim3(WG), lds, st, p, G1, G2, G3, (int)L, ws.dym, ws.rec, ws.tiles, ws.tile_base,
                       ws.part2, ws.pbuf, src[1], dst[1], mul);
    const int most = rw_extra(p, L), extra = most < RS_MAX_EXTRA ? most : RS_MAX_EXTRA;
    const RsArgs a{{src[0], src[1], src[2]}, {dst[0], dst[1], dst[2]}, mul, nwg, rw_piece(p, L), extra, K, cwgs, lines};
    const auto sum = !K ? rw_sum_kernel<C, false, false> : L < RW_SHARE_MIN_L ? rw_sum_kernel<C, true, false> : rw_sum_kernel<C, true, true>;
    hipLaunchKernelGGL(sum, dim3(cwgs + p.m1 + p.m3 + extra + p.m2 * per), dim3(RW_T), 0, st, p, ws, a, t0,
                       ws.dym, ws.pbuf, ws.l13);
    return hipGetLastError();
}

static inline hipError_t rw_bwd(const Params &p, const float *G1, const float *G2, const float *G3, int64_t L, const float *alpha, const float *go,
                                const float *t0, const float *const src[3], float *const dst[3], float mul, int K, float *lines,
                                const RowsWs &ws, hipStream_t st)
{
    switch (fast_config(p)) {
    case 2: return launch_rw_bwd<Cfg224R32, 128>(p, G1, G2, G3, L, alpha, go, t0, src, dst, mul, K, lines, ws, st);
    case 3: return launch_rw_bwd<Cfg224R64, 128>(p, G1, G2, G3, L, alpha, go, t0, src, dst, mul, K, lines, ws, st);
    case 4: return launch_rw_bwd<Cfg444R32, 128>(p, G1, G2, G3, L, alpha, go, t0, src, dst, mul, K, lines, ws, st);
    case 5: return launch_rw_bwd<Cfg444R64, 128>(p, G1, G2, G3, L, alpha, go, t0, src, dst, mul, K, lines, ws, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace tt
