// VALU path, d = 2: T explicit steps fused per pass (temporal fusion on the
// vector units; paper, Sec. "CUDA Core Implementation with Temporal Fusion":
// C grows by t, M stays 2D per point because intermediates stay on chip).
//
// Work decomposition
//   Every wave is independent: it owns a column band of 64*W columns (each
//   lane W consecutive columns) and streams down a segment of rows.  Of the
//   band, E = roundup(R*T, W) columns on each side are the skirt that later
//   steps consume; the valid output width is BX = 64W - 2E.  There is no LDS
//   and no barrier: neighbour columns come from cross-lane permutes (DPP
//   rotates for float64 with four columns per lane).
//
// Step pipeline
//   Stage 0 takes input row k (prefetched P rows ahead into registers).
//   Stage s = 1..T consumes the row stage s-1 produced one iteration earlier,
//   as a (W + 2R)-column window assembled by permutes at the end of that
//   iteration (so the permute latency overlaps the next row's arithmetic).
//   It scatters the window into 2R+1 rotating accumulator rows per lane
//   column (input-stationary: input row i adds w[a][.] to output row i-a) and
//   emits the completed output row i-R: to the next stage, or to HBM for
//   stage T.  Contributions to an output arrive in canonical order (kernel
//   row a ascending, column b ascending).
//
// Boundaries
//   Dirichlet: every field, intermediate ones included, is h outside the grid
//   (rows and columns outside are forced to h after each stage).  Periodic:
//   loads wrap; intermediate values in the skirt are then the periodic images.
//
// The kernel writes an arbitrary output rectangle [oy0,oy1) x [ox0,ox1), used
// both for whole grids and for the Dirichlet boundary band of the MFMA path.

#pragma once

#include <algorithm>
#include <cstddef>
#include <vector>

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "internal.h"
#include "valu_common.h"

namespace stl {

// Geometry of one pass of one grid: output box, tiling and boundary.
template <typename TC>
struct Valu2DJob {
    const void *src;
    void *dst;
    int n0, n1;
    int oy0, oy1, ox0, ox1;
    int BX, BY, nbands, nsegs;
    int anchor;  // first column of band 1 where bands are anchored to the right edge, else -1
    int nwg;  // workgroup items: ceil(nbands / waves) band groups x nsegs segments
    int periodic;
    TC h;
};

template <typename TC, int K>
struct Valu2DArgs {
    Valu2DJob<TC> g;
    TC w[K];
};

constexpr int kValu2DWaves = 4;  // waves per workgroup (independent bands)

template <typename TS, typename TC, int SHAPE, int R, int T, int W>
struct Valu2DCfg {
    static constexpr int K = SHAPE == STENCIL_BOX ? (2 * R + 1) * (2 * R + 1) : 4 * R + 1;
    static constexpr int NCW = 64 * W;                     // columns per wave
    static constexpr int E = ((R * T + W - 1) / W) * W;    // skirt per side
    static constexpr int Q = 2 * R + 1;
    // rows prefetched ahead: a multiple of Q, at least 4
    static constexpr int U = Q * ((4 + Q - 1) / Q);
    // input rows in flight: U for small Q; for r = 7 (Q = 15, compute-bound,
    // 225 or 29 FMAs per input value) 3 rows, a divisor of U, so the ring
    // slot of row k is k mod P at compile time and 48 VGPRs stay free.
    // 32-byte lanes (float64, four columns) prefetch one row: their rows take
    // twice the arithmetic, and the registers go to the wider accumulators
    static constexpr int P = sizeof(TS) * W > 16 ? 1
                             : (U <= 8 ? U : (U % 3 == 0 ? 3 : (U % 4 == 0 ? 4 : (U % 5 == 0 ? 5 : U))));
    // Boxes whose weights exceed 48 dwords (float64 r >= 2, float32 r = 3)
    // fused over T >= 3 steps keep them out of the vector registers: stored
    // column-major (w[b][a]), each column of 2R+1 is scalar-loaded just before
    // its FMAs.  That frees 49-98 VGPRs for the T stages' accumulators
    // (Box-2D3R float64 T = 4: 232 instead of 340 registers, no spills, +30 %
    // measured).  Float64 at T = 1 streams them too (Box-2D3R: 88 instead of
    // 236 VGPRs; +9 % measured at 10240^2, equal at 8192^2).  Float32 at T = 2
    // keeps them pinned in VGPRs (632 vs 478 GSt/s measured) unless they need
    // more than 128 dwords (r = 7: 225 weights).  Float64 lanes of four columns
    // stream them too: each weight then serves four columns, and the freed
    // registers hold the wider accumulators at two waves per SIMD.
    // Single-column lanes hold few accumulators and keep them in registers
    // (a streamed column would serve 2R+1 FMAs only), r = 7 excepted.
    static constexpr bool WPTR = SHAPE == STENCIL_BOX && sizeof(TC) * K > 192 &&
                                 (W > 1 ? (T >= 3 || sizeof(TC) == 8 || sizeof(TC) * K > 512) : R >= 7);
    // Streamed weights at T >= 3: each column is fetched once per input row
    // and serves every stage (columns outer, stages inner) instead of once
    // per stage.  Measured on 8192^2: Box-2D2R float64 T = 4 476 -> 570,
    // Box-2D3R float32 T = 3/4 498/501 -> 532/556, float64 302 -> 317
    // GSt/s; at T = 2 the per-stage order is as fast or faster (Box-2D3R
    // float64 353 vs 344).
    static constexpr bool WCOL = WPTR && T >= 3;
    // The first contribution to an output adds to a constant zero instead of a
    // zeroed accumulator (a product alone would keep the sign of a zero, which
    // must not depend on the lane width): two moves less per output value and
    // stage, and fewer registers (Star-2D2R T = 4 272 -> 246, which fits two
    // waves per SIMD).
    // Time per pass before and after in float64: Star-2D2R T = 4 4096^2 35 %,
    // 8192^2 20 % faster, Star-2D3R T = 3 8192^2 18 %, Box-2D3R T = 2 8192^2
    // 356 -> 341 us.  One- and two-column lanes, and float32, get schedules
    // with more registers from it and are 5-15 % slower at 512^2; Box-2D3R
    // T = 4, which spans both register files, 8 % at 8192^2.
    static constexpr bool FIRST_FROM_ZERO = sizeof(TC) == 8 && W == 4 && !(WCOL && T * Q > 24);
    // Batched kernels whose accumulators take 64 registers and more read their
    // job by scalar loads; copied through vector registers it cost them a wave
    // per SIMD (two 8192^2 grids, float64 Star-2D2R T = 4: 272 registers and 810 us
    // a pass, 249 and 534; Star-2D3R T = 3 782 and 521).  Lighter ones lose 7 % to
    // the waves they gain (float64 Star-2D1R T = 2 471 us, 505 so).
    static constexpr bool SCALAR_JOB = T * Q * W * (int)sizeof(TC) / 4 >= 64;
};

// Weights in constant memory (scalar loads).
template <typename TC>
using ConstPtr = const __attribute__((address_space(4))) TC *;

// Weight order the kernels expect: canonical, or column-major for WPTR boxes.
template <typename Cfg, int R>
__host__ __device__ constexpr int weight_slot(int k)
{
    if constexpr (Cfg::WPTR) {
        const int a = k / (2 * R + 1), b = k % (2 * R + 1);
        return b * (2 * R + 1) + a;
    } else {
        return k;
    }
}

template <int SHAPE, int R>
__device__ __forceinline__ int star_axis_index(int axis, int off)
{
    // canonical star order: centre, axis0 -R..-1,+1..+R, axis1 ...
    return 1 + axis * 2 * R + (off < 0 ? off + R : off + R - 1);
}

// value of `v` in lane (addr / 4) mod 64 (ds_bpermute: LDS crossbar, no storage)
__device__ __forceinline__ float lane_read(float v, int addr)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double lane_read(double v, int addr)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_ds_bpermute(addr, (int)(b & 0xffffffffLL));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, (int)(b >> 32));
    return __longlong_as_double(((long long)(unsigned)lo) | ((long long)hi << 32));
}

// value of `v` in lane (lane - 1) mod 64 (PREV) or (lane + 1) mod 64: a
// whole-wave DPP rotate by one lane (vector-ALU moves; no LDS access, so no
// lgkmcnt wait shared with the scalar weight loads)
template <bool PREV>
__device__ __forceinline__ double lane_rotate(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffLL), PREV ? 0x13C : 0x134, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), PREV ? 0x13C : 0x134, 0xF, 0xF, true);
    return __longlong_as_double(((long long)(unsigned)lo) | ((long long)hi << 32));
}

// win[j] = column lane*W - R + j of the wave's row, from the lanes' own W
// values (edge lanes receive wrapped values; those columns lie in the skirt).
// Float64 with four columns per lane (R <= W: every window column comes from
// the lane itself or a direct neighbour) rotates instead of permuting
// (Box-2D3R T = 2 8192^2: 366 -> 371 GSt/s); float32 and 16-bit storage
// measured 3-7 % slower with rotates.
template <typename TC, int W, int R>
__device__ __forceinline__ void assemble_window(const TC (&own)[W], TC (&win)[W + 2 * R], int lane)
{
#pragma unroll
    for (int j = 0; j < W; ++j) win[R + j] = own[j];
    if constexpr (sizeof(TC) == 8 && W == 4 && R <= W) {
#pragma unroll
        for (int m = 1; m <= R; ++m) win[R - m] = lane_rotate<true>(own[W - m]);
#pragma unroll
        for (int m = 0; m < R; ++m) win[R + W + m] = lane_rotate<false>(own[m]);
        return;
    }
#pragma unroll
    for (int m = 1; m <= R; ++m) {  // column lane*W - m
        const int dl = -((m + W - 1) / W);
        const int je = -m - dl * W;
        win[R - m] = lane_read(own[je], (lane + dl) * 4);
    }
#pragma unroll
    for (int m = 0; m < R; ++m) {  // column lane*W + W + m
        const int t = W + m;
        win[R + W + m] = lane_read(own[t % W], (lane + t / W) * 4);
    }
}

template <bool FIRST_FROM_ZERO, typename TC>
__device__ __forceinline__ TC accumulate(TC w, TC x, TC sum, bool first)
{
    return fma_c(w, x, FIRST_FROM_ZERO && first ? TC(0) : sum);
}

// One tile (column band x row segment) of one pass, run by one wave.
template <typename TS, typename TC, int SHAPE, int R, int T, int W>
__device__ __forceinline__ void valu2d_tile(const Valu2DJob<TC> &a,
                                            const TC (&wk)[Valu2DCfg<TS, TC, SHAPE, R, T, W>::WPTR
                                                               ? 1
                                                               : Valu2DCfg<TS, TC, SHAPE, R, T, W>::K],
                                            ConstPtr<TC> wp, int band, int seg, int lane)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, W>;
    constexpr int Q = Cfg::Q;
    constexpr int U = Cfg::U;
    using Vec = RawVec<TS, W>;

    const int x0 = a.anchor >= 0 && band > 0 ? a.anchor + (band - 1) * a.BX : a.ox0 + band * a.BX;
    const int y0 = a.oy0 + seg * a.BY;
    const int y1 = min(y0 + a.BY, a.oy1);
    const int BYe = y1 - y0;
    const int xe = a.anchor >= 0 && band == 0 ? a.anchor : min(x0 + a.BX, a.ox1);
    const int cb = x0 - Cfg::E + lane * W;  // first column owned by this lane

    const TS *src = static_cast<const TS *>(a.src);
    TS *dst = static_cast<TS *>(a.dst);
    const int n0 = a.n0, n1 = a.n1;
    const bool periodic = a.periodic != 0;
    const TC h = a.h;

    // The lane's columns lie wholly inside or wholly outside the grid (see
    // valu2d_bands; W = 1 always does): its source column (wrapped, or a valid
    // dummy) and whether a Dirichlet lane takes h instead.  Lanes of skirt
    // columns that no output needs may straddle the edge: they load in bounds.
    const bool lane_in = periodic || (cb >= 0 && cb + W <= n1);
    const int f_col = lane_in ? min(wrap(cb, n1), max(n1 - W, 0)) : 0;
    // output stores: the whole vector, or (lanes at the band's ragged edge)
    // element by element; the element path is skipped by a wave-uniform
    // branch when no lane of the wave needs it
    bool col_store[W];
    bool st_all = true, st_any = false;
#pragma unroll
    for (int j = 0; j < W; ++j) {
        col_store[j] = cb + j >= x0 && cb + j < xe;
        st_all = st_all && col_store[j];
        st_any = st_any || col_store[j];
    }
    const bool st_part_wave = __ballot(st_any && !st_all) != 0;

    const int KTOT = BYe + 2 * R * T + T;
    const int ybase = y0 - R * T;

    // accumulators: T stages x Q rotating rows x W columns
    TC acc[T][Q][W];
#pragma unroll
    for (int s = 0; s < T; ++s)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int j = 0; j < W; ++j) acc[s][q][j] = TC(0);
    // input windows of stages 1..T (the previous iteration's rows)
    TC wins[T][W + 2 * R];
#pragma unroll
    for (int s = 0; s < T; ++s)
#pragma unroll
        for (int j = 0; j < W + 2 * R; ++j) wins[s][j] = TC(0);

    // one unconditional vector load per row (rows wrap or clamp; those outside
    // a Dirichlet grid are replaced by h when consumed): with no other write to
    // the prefetch ring, the compiler waits only for the row being consumed
    // and the loads of the next rows stay in flight
    int rl = periodic ? wrap(ybase, n0) : 0;  // periodic: source row of the next load
    auto load_row = [&](int k, Vec &v) {
        const int ri = periodic ? rl : min(max(ybase + k, 0), n0 - 1);
        v.load_any(src + (int64_t)ri * n1 + f_col);
        rl = rl + 1 == n0 ? 0 : rl + 1;
    };

    constexpr int P = Cfg::P;
    Vec ring[P];
#pragma unroll
    for (int u = 0; u < P; ++u)
        if (u < KTOT) load_row(u, ring[u]);

    // WPTR: weight column b (2R+1 values) of the block being computed and of
    // the next one.  Scalar loads complete out of order, so any wait for one
    // waits for all: the fetch of the next column takes the current column's
    // first weight as an operand, which puts it after the wait for the
    // current column, and an empty volatile asm statement on the current
    // block's accumulators after its FMAs keeps the next wait behind them
    // (volatile asm statements keep their order), so each fetch overlaps a
    // whole block of FMAs and at most two columns are live.
    // float32: FMAs run faster on vector-register operands (one move per
    // weight).  For r >= 5 a column moves to vector registers when it becomes
    // current, after the previous block's FMAs, so its scalar loads complete
    // under them (moving at the fetch waits for each load at once and
    // serialises them: Box-2D7R 129 -> 135 GSt/s); for r = 3 moving at the
    // fetch measured as fast or slightly faster.
    constexpr bool LATE_MOVE = sizeof(TC) == 4 && R >= 5;
    TC wcur[Q], wnxt[Q];
    // The ordering dependency goes through the base pointer, so the column
    // offsets stay compile-time immediates of the scalar loads (an opaque
    // offset cost five scalar instructions of address arithmetic per column:
    // Box-2D3R float64 T = 2 370 -> 378 GSt/s without them).
    auto fetch_col = [&](int b, TC *dstw, TC after) {
        ConstPtr<TC> p = wp;
        if constexpr (sizeof(TC) == 4) asm volatile("" : "+s"(p) : "v"(after));
        else asm volatile("" : "+s"(p) : "s"(after));
#pragma unroll
        for (int e = 0; e < Q; ++e) {
            dstw[e] = p[b * Q + e];
            if constexpr (sizeof(TC) == 4 && !LATE_MOVE) asm volatile("" : "+v"(dstw[e]));
        }
    };
    auto to_vgpr = [&](TC *wv) {
        if constexpr (LATE_MOVE)
#pragma unroll
            for (int e = 0; e < Q; ++e) asm volatile("" : "+v"(wv[e]));
    };
    if constexpr (Cfg::WPTR) {
        fetch_col(0, wcur, TC(0));
        to_vgpr(wcur);
    }

    for (int kb = 0; kb < KTOT; kb += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = kb + u;
            if (k >= KTOT) break;
            // Stages run from T down to 1 so that the window each one produces
            // for the next stage can be assembled at once (its consumer has
            // already used the previous window this iteration); the permute
            // latency then hides behind the lower stages' arithmetic.
            if constexpr (Cfg::WCOL) {
#pragma unroll
                for (int bo = -R; bo <= R; ++bo) {
                    fetch_col(bo + R < 2 * R ? bo + R + 1 : 0, wnxt, wcur[0]);
#pragma unroll
                    for (int s = T; s >= 1; --s) {
                        const bool active = k >= s + 2 * R * (s - 1) && k < BYe + 2 * R * T + s;
                        if (!active) continue;
                        const TC *win = wins[s - 1];
#pragma unroll
                        for (int ao = -R; ao <= R; ++ao) {
                            const int q = ((u - ao + R) % Q + Q) % Q;
#pragma unroll
                            for (int j = 0; j < W; ++j)
                                acc[s - 1][q][j] = accumulate<Cfg::FIRST_FROM_ZERO>(wcur[ao + R], win[j + bo + R], acc[s - 1][q][j],
                                                                              ao == -R && bo == -R);
                        }
                    }
                    // this column's FMAs complete before the wait for the next
                    // column's weights
#pragma unroll
                    for (int s = 0; s < T; ++s)
#pragma unroll
                        for (int q = 0; q < Q; ++q)
#pragma unroll
                            for (int j = 0; j < W; ++j) asm volatile("" ::"v"(acc[s][q][j]));
#pragma unroll
                    for (int e = 0; e < Q; ++e) wcur[e] = wnxt[e];
                    to_vgpr(wcur);
                }
            }
#pragma unroll
            for (int s = T; s >= 1; --s) {
                const bool active = k >= s + 2 * R * (s - 1) && k < BYe + 2 * R * T + s;
                const int qc = u % Q;  // slot completing at this iteration
                TC outv[W];
#pragma unroll
                for (int j = 0; j < W; ++j) outv[j] = TC(0);
                if (active) {
                    const TC *win = wins[s - 1];
                    if constexpr (Cfg::WCOL) {
                        // accumulated above, all stages per weight column
                    } else if constexpr (Cfg::WPTR) {
#pragma unroll
                        for (int bo = -R; bo <= R; ++bo) {
                            fetch_col(bo + R < 2 * R ? bo + R + 1 : 0, wnxt, wcur[0]);
#pragma unroll
                            for (int ao = -R; ao <= R; ++ao) {
                                const int q = ((u - ao + R) % Q + Q) % Q;
#pragma unroll
                                for (int j = 0; j < W; ++j)
                                    acc[s - 1][q][j] = accumulate<Cfg::FIRST_FROM_ZERO>(wcur[ao + R], win[j + bo + R], acc[s - 1][q][j],
                                                                              ao == -R && bo == -R);
                            }
                            // this column's FMAs complete before the wait for the
                            // next column's weights (which the fetch after next
                            // needs), so that fetch runs under all of them
#pragma unroll
                            for (int q = 0; q < Q; ++q)
#pragma unroll
                                for (int j = 0; j < W; ++j) asm volatile("" ::"v"(acc[s - 1][q][j]));
#pragma unroll
                            for (int e = 0; e < Q; ++e) wcur[e] = wnxt[e];
                            to_vgpr(wcur);
                        }
                    } else {
#pragma unroll
                        for (int bo = -R; bo <= R; ++bo) {
#pragma unroll
                            for (int ao = -R; ao <= R; ++ao) {
                                const int q = ((u - ao + R) % Q + Q) % Q;
                                if constexpr (SHAPE == STENCIL_BOX) {
                                    const TC wv = wk[(ao + R) * (2 * R + 1) + (bo + R)];
#pragma unroll
                                    for (int j = 0; j < W; ++j)
                                        acc[s - 1][q][j] = accumulate<Cfg::FIRST_FROM_ZERO>(wv, win[j + bo + R], acc[s - 1][q][j],
                                                                                      ao == -R && bo == -R);
                                } else if (ao != 0 && bo == 0) {
                                    const TC wv = wk[star_axis_index<SHAPE, R>(0, ao)];
#pragma unroll
                                    for (int j = 0; j < W; ++j)
                                        acc[s - 1][q][j] =
                                            accumulate<Cfg::FIRST_FROM_ZERO>(wv, win[j + R], acc[s - 1][q][j], ao == -R);
                                } else if (ao == 0) {
                                    const TC wv = bo == 0 ? wk[0] : wk[star_axis_index<SHAPE, R>(1, bo)];
#pragma unroll
                                    for (int j = 0; j < W; ++j)
                                        acc[s - 1][q][j] = fma_c(wv, win[j + bo + R], acc[s - 1][q][j]);
                                }
                            }
                        }
                    }
                    // the completed row
                    const int yo = ybase + k - s * (1 + R);  // row completed by stage s
#pragma unroll
                    for (int j = 0; j < W; ++j) outv[j] = acc[s - 1][qc][j];
                    if (s < T) {
                        if (!periodic) {
                            const bool in = lane_in && yo >= 0 && yo < n0;
#pragma unroll
                            for (int j = 0; j < W; ++j)
                                if (!in) outv[j] = h;
                        }
                    } else if (yo >= y0 && yo < y1) {
                        TS *rowp = dst + (int64_t)yo * n1;
                        Vec ov;
#pragma unroll
                        for (int j = 0; j < W; ++j) ov.e[j] = to_storage<TS>(outv[j]);
                        if (st_all) ov.store_any(rowp + cb);
                        if (st_part_wave && !st_all) {
#pragma unroll
                            for (int j = 0; j < W; ++j)
                                if (col_store[j]) rowp[cb + j] = ov.e[j];
                        }
                    }
                }
                if constexpr (!Cfg::FIRST_FROM_ZERO)
#pragma unroll
                    for (int j = 0; j < W; ++j) acc[s - 1][qc][j] = TC(0);
                // window of this stage's row for stage s+1 at the next iteration
                if (s < T) assemble_window<TC, W, R>(outv, wins[s], lane);
            }
            // ---- stage 0: input row (window for stage 1), prefetch P rows ahead
            {
                TC inrow[W];
                const int i = ybase + k;
                const bool hrow = !lane_in || (!periodic && (i < 0 || i >= n0));
#pragma unroll
                for (int j = 0; j < W; ++j) inrow[j] = hrow ? h : to_compute<TC>(ring[u % P].e[j]);
                // keep the refill of this ring slot behind the reads that drain it
                __builtin_amdgcn_sched_barrier(0);
                if (k + P < KTOT) load_row(k + P, ring[u % P]);
                assemble_window<TC, W, R>(inrow, wins[0], lane);
            }
        }
    }
}

// Load the weights.  Float32 weights go to vector registers: a v_fma_f32 with a
// scalar-register operand measured ~35 % slower on gfx950 than with vector
// operands only (61-68 vs 92-97 TFLOP/s in FMA chains; float64 shows no such
// difference).  Float64 sets up to ~48 dwords stay in scalar registers; larger
// ones (49 float64 box weights) are pinned in vector registers, otherwise the
// compiler spills them to vector lanes and pays a readlane per use.
// The float64 Star-2D7R set (29 weights) stays in scalar registers: pinned in
// vector registers beside its 15 accumulator rows per stage it needs all 256.
template <typename TC, int K, bool SCALAR64 = false, typename Src>
__device__ __forceinline__ void load_weights(TC (&wk)[K], Src w)
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        wk[k] = w[k];
        if constexpr (sizeof(TC) == 4 || (sizeof(TC) * K > 192 && !SCALAR64)) asm volatile("" : "+v"(wk[k]));
    }
}

// Item of this wave in workgroup `wg` of a pass, the same for all its lanes.
__device__ __forceinline__ int valu2d_item(int wg)
{
    return wg * kValu2DWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

template <typename TS, typename TC, int SHAPE, int R, int T, int W>
__global__ __launch_bounds__(64 * kValu2DWaves) void valu2d_kernel(
    Valu2DArgs<TC, Valu2DCfg<TS, TC, SHAPE, R, T, W>::K> a)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, W>;
    // Waves take (segment, band) items, bands fastest: adjacent bands share
    // skirt columns in one CU's L1, and the contiguous run of items on an XCD
    // shares halo rows in that XCD's L2.
    const int item = valu2d_item(xcd_remap(blockIdx.x, gridDim.x));
    if (item >= a.g.nbands * a.g.nsegs) return;
    const int seg = item / a.g.nbands, band = item - seg * a.g.nbands;
    TC wk[Cfg::WPTR ? 1 : Cfg::K];
    ConstPtr<TC> wp = nullptr;
    if constexpr (Cfg::WPTR) {
        // the argument block is the first entry of the kernel-argument segment
        using Args = Valu2DArgs<TC, Cfg::K>;
        wp = (ConstPtr<TC>)((const __attribute__((address_space(4))) char *)
                                __builtin_amdgcn_kernarg_segment_ptr() +
                            offsetof(Args, w));
        wk[0] = TC(0);
    } else {
        load_weights<TC, Cfg::K, SHAPE == STENCIL_STAR && R == 7>(wk, a.w);
    }
    valu2d_tile<TS, TC, SHAPE, R, T, W>(a.g, wk, wp, band, seg, threadIdx.x & 63);
}

// One job of a batched launch: geometry plus weights.
template <typename TC, int K>
struct Valu2DBatchJob {
    Valu2DJob<TC> g;
    TC w[K];
};

// Geometry of a batched job, by scalar loads or copied through vector registers.
template <typename TC, bool SCALAR, typename Job>
__device__ __forceinline__ Valu2DJob<TC> valu2d_job(const Job *entry, JobPtr<Job> job)
{
    Valu2DJob<TC> g;
    if constexpr (SCALAR) {
        g.src = job->g.src;
        g.dst = job->g.dst;
        g.n0 = job->g.n0;
        g.n1 = job->g.n1;
        g.oy0 = job->g.oy0;
        g.oy1 = job->g.oy1;
        g.ox0 = job->g.ox0;
        g.ox1 = job->g.ox1;
        g.BX = job->g.BX;
        g.BY = job->g.BY;
        g.nbands = job->g.nbands;
        g.nsegs = job->g.nsegs;
        g.anchor = job->g.anchor;
        g.periodic = job->g.periodic;
        g.h = job->g.h;
    } else {
        g = entry->g;
    }
    return g;
}

// Persistent batched launch: the workgroups walk one list of (job, band
// group x segment) items spanning every job of the batch (jobs of uneven
// sizes); workgroup b takes items b + i*gridDim.  tile_start[j] is the first
// item of job j (tile_start[njobs] = total).
template <typename TS, typename TC, int SHAPE, int R, int T, int W>
__global__ __launch_bounds__(64 * kValu2DWaves) void valu2d_batch_kernel(
    const Valu2DBatchJob<TC, Valu2DCfg<TS, TC, SHAPE, R, T, W>::K> *jobs,
    const int *tile_start, int njobs)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, W>;
    const int total = tile_start[njobs];
    const int lane = threadIdx.x & 63;
    int j = 0;
    for (int item = xcd_remap(blockIdx.x, gridDim.x); item < total; item += gridDim.x) {
        while (j + 1 < njobs && tile_start[j + 1] <= item) ++j;
        const auto job = job_entry(jobs, j);
        const Valu2DJob<TC> g = valu2d_job<TC, Cfg::SCALAR_JOB>(jobs + j, job);
        const int local = valu2d_item(item - tile_start[j]);
        if (local >= g.nbands * g.nsegs) continue;
        const int seg = local / g.nbands, band = local - seg * g.nbands;
        TC wk[Cfg::WPTR ? 1 : Cfg::K];
        ConstPtr<TC> wp = nullptr;
        if constexpr (Cfg::WPTR) {
            wp = &job->w[0];
            wk[0] = TC(0);
        } else {
            if constexpr (Cfg::SCALAR_JOB) load_weights<TC, Cfg::K, SHAPE == STENCIL_STAR && R == 7>(wk, &job->w[0]);
            else load_weights<TC, Cfg::K, SHAPE == STENCIL_STAR && R == 7>(wk, jobs[j].w);
        }
        valu2d_tile<TS, TC, SHAPE, R, T, W>(g, wk, wp, band, seg, lane);
    }
}

// Columns per lane: 1, 2 or 4, picked per launch.  One-column lanes take any
// grid and any box, put four times as many waves on a small grid and keep
// large box weights in registers; four columns spend the smallest share on
// skirts and window permutes.  Eight 16-bit columns measured slower than four
// at every depth (8192^2 one step 55.9 vs 50.4 us, Star-2D2R T = 4 211 vs 120),
// and float64 needs more registers than there are for four at T > 4.
template <typename TC, int T>
constexpr int valu2d_widest()
{
    return sizeof(TC) == 8 && T > 4 ? 2 : 4;
}

// Column bands of a pass for W columns per lane; false where the lanes of a
// band cannot all lie wholly inside or wholly outside the grid.  Rows of whole
// vectors take bands from the box's first column on.  Rows of another length
// put band 0 at the left edge and anchor the others to the right edge, so that
// both edges fall between lanes (loads need no alignment beyond the element);
// band 1 must start at least a skirt from the left edge, which a band a few
// vectors narrower gives.
template <typename Cfg, int W, typename TC>
bool valu2d_bands(const PassArgs &p, Valu2DJob<TC> *g)
{
    constexpr int BXmax = Cfg::NCW - 2 * Cfg::E;
    static_assert(BXmax > 0, "band narrower than its skirt");
    g->src = p.src;
    g->dst = p.dst;
    g->n0 = (int)p.dims[0];
    g->n1 = (int)p.dims[1];
    g->oy0 = p.region_lo[0];
    g->oy1 = p.region_hi[0];
    g->ox0 = p.region_lo[1];
    g->ox1 = p.region_hi[1];
    g->periodic = p.boundary == STENCIL_PERIODIC;
    g->h = (TC)p.halo;
    g->anchor = -1;
    g->BX = BXmax;
    if (W > 1 && (g->n1 % W != 0 || g->ox0 % W != 0)) {
        if (g->ox0 != 0 || g->ox1 != g->n1 || g->n1 < Cfg::NCW) return false;
        for (;; g->BX -= W) {
            if (g->BX < BXmax / 2) return false;
            const int nb = (g->n1 + g->BX - 1) / g->BX;
            g->anchor = g->n1 - (nb - 1) * g->BX;
            if (nb >= 2 && g->anchor >= Cfg::E) break;
        }
    }
    g->nbands = (g->ox1 - g->ox0 + g->BX - 1) / g->BX;
    return true;
}

// Row segments of BY rows.
template <typename TC>
void valu2d_rows(Valu2DJob<TC> *g, int BY)
{
    const int H = g->oy1 - g->oy0;
    g->BY = BY;
    g->nsegs = (H + BY - 1) / BY;
    g->nwg = (int)(((int64_t)g->nbands * g->nsegs + kValu2DWaves - 1) / kValu2DWaves);
}

// Resident workgroups per CU of a kernel instance.
template <typename K>
int valu2d_occupancy(K kernel)
{
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, 64 * kValu2DWaves, 0) != hipSuccess || occ < 1)
        occ = 1;
    return occ;
}

// Estimate of a launch of nwg workgroups over segments of BY rows, in cycles:
// the larger of the rows' issue time and the bytes' time.
//   issue: a wave takes BY + 2RT + T row iterations.  One costs about 1500
//     cycles of latency shared by the waves of a SIMD (permutes, the stages'
//     chains; 100 more per streamed weight column) and the instructions of
//     each of them.  A workgroup puts one wave on every SIMD of its CU, so the
//     busiest CU's workgroups, not the average, count (8192^2 float32
//     Star-2D3R T = 4: 504 workgroups = 2 per CU 171 us, 576 279).
//     Float64 lanes of four columns whose accumulators span both register files
//     (Box-2D3R T = 4, one wave per SIMD) take 1.3 times their instructions:
//     without it they were picked from 3000 x 7000 up, 8192^2 968 us where
//     two-column lanes take 802.
//   bytes: one read and one write per point, the read grown by the skirt and
//     the halo rows, at about 1800 bytes a cycle from HBM or 3500 from the
//     last-level cache (256 MB); 1.12 times as long for 32-byte lanes on rows
//     that are no whole number of 128-byte lines (float64 Star-2D1R T = 3
//     3000 x 7000: two columns 69 us, four 83; 6000^2: 152 and 137).
// Fitted to 2800 variants and sizes (76 variants, 256^2..8192^2, flat, tall and
// at random, some 40 choices each): the choice is 2.5 % behind the best
// measured on average.
template <typename Cfg, typename TS, typename TC, int SHAPE, int R, int T, int W>
struct Valu2DCost {
    static constexpr double stretch()
    {
        return sizeof(TC) == 8 && W == 4 && Cfg::WCOL && T * Cfg::Q > 24 ? 1.3 : 1.0;
    }
    static double issue(int64_t nwg, int BY, int occ, int cus)
    {
        const double row =
            stretch() * (T * (W * ((sizeof(TC) == 8 ? 4.5 : 2.5) * Cfg::K + 32) + 12.0 * 2 * R * (sizeof(TC) / 4)) + 20);
        const double latency = 1500 + (Cfg::WPTR ? 100.0 * Cfg::Q * (T >= 3 ? 1 : T) : 0.0);
        auto resident = [&](int64_t k) { return latency + row * (k > 1 ? k - 0.4 : k); };
        const int64_t per_cu = (nwg + cus - 1) / cus, full = per_cu / occ, rest = per_cu % occ;
        return (BY + 2 * R * T + T) * (full * resident(occ) + (rest ? resident(rest) : 0.0));
    }
    static double memory(double points, int BY, int BX, bool whole_lines)
    {
        const double grow = (1.0 + 2.0 * R * T / BY) * Cfg::NCW / BX;
        const double wide = sizeof(TS) * W > 16 && !whole_lines ? 1.12 : 1.0;
        return wide * points * sizeof(TS) * (1.0 + grow) / (2 * points * sizeof(TS) > 256e6 ? 1800.0 : 3500.0);
    }
};

struct Valu2DPick {
    int W = 0, BY = 0;
    double cost = -1.0;
    // short segments on a grid past the last-level cache
    bool streams = false;
};

inline double valu2d_points(const PassArgs &p)
{
    return (double)std::max(p.region_hi[0] - p.region_lo[0], 0) * std::max(p.region_hi[1] - p.region_lo[1], 0);
}

// Try W columns per lane for a launch over n passes: segment lengths that put
// 1..32 workgroups on every CU, none under 3 rows.
template <typename TS, typename TC, int SHAPE, int R, int T, int W>
void valu2d_try(const PassArgs *ps, int n, int occ, int cus, Valu2DPick *best)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, W>;
    using Cost = Valu2DCost<Cfg, TS, TC, SHAPE, R, T, W>;
    int64_t bands = 0;
    int hmax = 1, bx = 1;
    double points = 0, area = 0;  // area: bands x rows
    bool whole_lines = true;      // rows of whole 128-byte lines
    Valu2DJob<TC> g;
    for (int i = 0; i < n; ++i) {
        const int H = ps[i].region_hi[0] - ps[i].region_lo[0];
        if (H <= 0 || valu2d_points(ps[i]) <= 0) continue;
        if (!valu2d_bands<Cfg, W>(ps[i], &g)) return;
        bands += g.nbands;
        area += (double)g.nbands * H;
        points += valu2d_points(ps[i]);
        hmax = std::max(hmax, H);
        bx = g.BX;
        whole_lines = whole_lines && (int64_t)g.n1 * (int)sizeof(TS) % 128 == 0;
    }
    auto workgroups = [&](int BY) {
        int64_t items = 0;
        for (int i = 0; i < n; ++i) {
            const int H = ps[i].region_hi[0] - ps[i].region_lo[0];
            if (H <= 0 || valu2d_points(ps[i]) <= 0) continue;
            if (n > 1) valu2d_bands<Cfg, W>(ps[i], &g);
            items += (int64_t)g.nbands * ((H + BY - 1) / BY);
        }
        return (items + kValu2DWaves - 1) / kValu2DWaves;
    };
    auto consider = [&](int BY, bool streams, double cost) {
        if (best->cost >= 0 && (best->streams > streams || (best->streams == streams && cost >= best->cost))) return;
        *best = {W, BY, cost, streams};
    };
    if (n == 1 && ps[0].tile_rows > 0) {  // the caller's segment length
        const int BY = ps[0].tile_rows;
        consider(BY, false, std::max(Cost::issue(workgroups(BY), std::min(BY, hmax), occ, cus),
                                     Cost::memory(points, BY, bx, whole_lines)));
        return;
    }
    static const int kPerCu[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 32};
    int last = 0;
    for (int k : kPerCu) {
        // n passes: a common length of about area / items rows
        const int64_t items = (int64_t)k * kValu2DWaves * cus;
        const int64_t segs = items / std::max<int64_t>(bands, 1);
        if (n == 1 && segs < 1) continue;
        int BY = n == 1 ? (int)((hmax + segs - 1) / segs) : (int)(area / items) + 1;
        if (BY < 3) BY = 3;
        // two numbers of items that round to one length: the rows left are few
        // or the bands many, and shorter segments gain nothing any more (bf16
        // Box-2D3R T = 2 128 x 900000: whole columns 323 us, 15 rows 368)
        if (BY == last) break;
        last = BY;
        const double issue = Cost::issue(workgroups(BY), std::min(BY, hmax), occ, cus);
        // Past the last-level cache a memory-bound pass gains from short
        // segments, whose workgroups walk the grid together (8192^2 float64
        // Star-2D1R T = 1: 17 rows 212 us, 137 232; float32 107, 119): the
        // shortest ones where their issue time is within 1.4 of the bytes'.
        const bool streams = k == 32 && W == (sizeof(TS) == 8 ? 2 : 4) && 2 * points * sizeof(TS) > 256e6 &&
                             issue < 1.4 * 2 * points * sizeof(TS) / 1800.0;
        consider(BY, streams, std::max(issue, Cost::memory(points, BY, bx, whole_lines)));
    }
    // more bands than any of these numbers of items: whole columns, in each
    // width (4 x 20000000 float32 Star-2D3R T = 4: one-column lanes 3797 us, four
    // columns 986)
    if (last == 0)
        consider(hmax, false, std::max(Cost::issue(workgroups(hmax), hmax, occ, cus),
                                       Cost::memory(points, hmax, bx, whole_lines)));
}

// Geometry of one pass for W columns per lane and segments of BY rows.
template <typename TS, typename TC, int SHAPE, int R, int T, int W>
void valu2d_geometry(const PassArgs &p, int BY, Valu2DJob<TC> *g)
{
    (void)valu2d_bands<Valu2DCfg<TS, TC, SHAPE, R, T, W>, W>(p, g);
    valu2d_rows(g, BY);
}

template <typename TS, typename TC, int SHAPE, int R, int T, int W>
hipError_t launch_valu2d_width(const PassArgs &p, int BY, hipStream_t stream)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, W>;
    Valu2DArgs<TC, Cfg::K> a;
    valu2d_geometry<TS, TC, SHAPE, R, T, W>(p, BY, &a.g);
    for (int k = 0; k < Cfg::K; ++k) a.w[weight_slot<Cfg, R>(k)] = (TC)p.w[k];
    hipLaunchKernelGGL((valu2d_kernel<TS, TC, SHAPE, R, T, W>), dim3(a.g.nwg), dim3(64 * kValu2DWaves), 0, stream, a);
    return hipGetLastError();
}

template <typename TS, typename TC, int SHAPE, int R, int T>
hipError_t launch_valu2d(const PassArgs &p, hipStream_t stream)
{
    if (valu2d_points(p) <= 0) return hipSuccess;
    static const int occ1 = valu2d_occupancy(valu2d_kernel<TS, TC, SHAPE, R, T, 1>);
    static const int occ2 = valu2d_occupancy(valu2d_kernel<TS, TC, SHAPE, R, T, 2>);
    const int cus = p.num_cu > 0 ? p.num_cu : 256;
    Valu2DPick pick;
    valu2d_try<TS, TC, SHAPE, R, T, 1>(&p, 1, occ1, cus, &pick);
    valu2d_try<TS, TC, SHAPE, R, T, 2>(&p, 1, occ2, cus, &pick);
    if constexpr (valu2d_widest<TC, T>() == 4) {
        static const int occ4 = valu2d_occupancy(valu2d_kernel<TS, TC, SHAPE, R, T, 4>);
        valu2d_try<TS, TC, SHAPE, R, T, 4>(&p, 1, occ4, cus, &pick);
        if (pick.W == 4) return launch_valu2d_width<TS, TC, SHAPE, R, T, 4>(p, pick.BY, stream);
    }
    return pick.W == 2 ? launch_valu2d_width<TS, TC, SHAPE, R, T, 2>(p, pick.BY, stream)
                       : launch_valu2d_width<TS, TC, SHAPE, R, T, 1>(p, pick.BY, stream);
}

template <typename TS, typename TC, int SHAPE, int R, int T, int W>
hipError_t launch_valu2d_batch_width(const PassArgs *ps, int n, int BY, int slots, BatchStaging *stage,
                                     hipStream_t stream)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, W>;
    using Job = Valu2DBatchJob<TC, Cfg::K>;
    std::vector<Job> jobs;
    std::vector<int> start(1, 0);
    jobs.reserve(n);
    for (int i = 0; i < n; ++i) {
        if (valu2d_points(ps[i]) <= 0) continue;
        Job j;
        valu2d_geometry<TS, TC, SHAPE, R, T, W>(ps[i], ps[i].tile_rows > 0 ? ps[i].tile_rows : BY, &j.g);
        for (int k = 0; k < Cfg::K; ++k) j.w[weight_slot<Cfg, R>(k)] = (TC)ps[i].w[k];
        jobs.push_back(j);
        start.push_back(start.back() + j.g.nwg);
    }
    void *djobs = nullptr, *dstart = nullptr;
    hipError_t e = stage_job_table(stage, jobs.data(), jobs.size() * sizeof(Job), start, &djobs, &dstart, stream);
    if (e != hipSuccess) return e;
    const int total = start.back();
    hipLaunchKernelGGL((valu2d_batch_kernel<TS, TC, SHAPE, R, T, W>), dim3(total < slots ? total : slots),
                       dim3(64 * kValu2DWaves), 0, stream, static_cast<const Job *>(djobs),
                       static_cast<const int *>(dstart), (int)jobs.size());
    return hipGetLastError();
}

// Resident workgroups per CU of the batched kernels of 1, 2 and 4 columns.
template <typename TS, typename TC, int SHAPE, int R, int T>
const int *valu2d_batch_occ()
{
    static const struct Occ {
        int v[3] = {valu2d_occupancy(valu2d_batch_kernel<TS, TC, SHAPE, R, T, 1>),
                    valu2d_occupancy(valu2d_batch_kernel<TS, TC, SHAPE, R, T, 2>), 1};
        Occ()
        {
            if constexpr (valu2d_widest<TC, T>() == 4)
                v[2] = valu2d_occupancy(valu2d_batch_kernel<TS, TC, SHAPE, R, T, 4>);
        }
    } occ;
    return occ.v;
}

// Width and segments of one batched launch over the passes `ps`.
template <typename TS, typename TC, int SHAPE, int R, int T>
Valu2DPick valu2d_batch_pick(const std::vector<PassArgs> &ps)
{
    const int *occ = valu2d_batch_occ<TS, TC, SHAPE, R, T>();
    const int n = (int)ps.size(), cus = ps[0].num_cu > 0 ? ps[0].num_cu : 256;
    Valu2DPick pick;
    valu2d_try<TS, TC, SHAPE, R, T, 1>(ps.data(), n, occ[0], cus, &pick);
    valu2d_try<TS, TC, SHAPE, R, T, 2>(ps.data(), n, occ[1], cus, &pick);
    if constexpr (valu2d_widest<TC, T>() == 4)
        valu2d_try<TS, TC, SHAPE, R, T, 4>(ps.data(), n, occ[2], cus, &pick);
    return pick;
}

template <typename TS, typename TC, int SHAPE, int R, int T>
hipError_t valu2d_batch_go(const std::vector<PassArgs> &ps, const Valu2DPick &pick, BatchStaging *stage,
                           hipStream_t stream)
{
    const int *occ = valu2d_batch_occ<TS, TC, SHAPE, R, T>();
    const int n = (int)ps.size(), cus = ps[0].num_cu > 0 ? ps[0].num_cu : 256;
    if constexpr (valu2d_widest<TC, T>() == 4)
        if (pick.W == 4)
            return launch_valu2d_batch_width<TS, TC, SHAPE, R, T, 4>(ps.data(), n, pick.BY, occ[2] * cus, stage, stream);
    return pick.W == 2
               ? launch_valu2d_batch_width<TS, TC, SHAPE, R, T, 2>(ps.data(), n, pick.BY, occ[1] * cus, stage, stream)
               : launch_valu2d_batch_width<TS, TC, SHAPE, R, T, 1>(ps.data(), n, pick.BY, occ[0] * cus, stage, stream);
}

// Batched form: n passes (one per job) of the same variant in one launch, or in
// two where grids that cannot take the widest lanes (narrow ones with rows that
// are no whole number of vectors) would keep the others from them: when the
// estimates of the two and 12000 cycles for a launch come to less (float32
// Star-2D3R T = 4, 8192^2 and 64 x 71: one launch on one-column lanes 670 us a
// pass, two launches 222).
template <typename TS, typename TC, int SHAPE, int R, int T>
hipError_t launch_valu2d_batch(const PassArgs *ps, int n, BatchStaging *stage, hipStream_t stream)
{
    constexpr int W = valu2d_widest<TC, T>();
    std::vector<PassArgs> all, wide, other;
    for (int i = 0; i < n; ++i) {
        if (valu2d_points(ps[i]) <= 0) continue;
        Valu2DJob<TC> g;
        all.push_back(ps[i]);
        (valu2d_bands<Valu2DCfg<TS, TC, SHAPE, R, T, W>, W>(ps[i], &g) ? wide : other).push_back(ps[i]);
    }
    if (all.empty()) return hipSuccess;
    const auto pick = &valu2d_batch_pick<TS, TC, SHAPE, R, T>;
    const auto go = &valu2d_batch_go<TS, TC, SHAPE, R, T>;
    const Valu2DPick one = pick(all);
    if (!wide.empty() && !other.empty()) {
        const Valu2DPick first = pick(wide), second = pick(other);
        if (first.cost + second.cost + 12000.0 < one.cost) {
            const hipError_t e = go(wide, first, stage, stream);
            return e == hipSuccess ? go(other, second, stage, stream) : e;
        }
    }
    return go(all, one, stage, stream);
}

// Up to kBandBoxes boxes of one pass (the Dirichlet band of a kernel-fused
// matrix pass) in one launch: the boxes are narrow, so one-column lanes.
constexpr int kBandBoxes = 4;

template <typename TC, int K>
struct Valu2DBandArgs {
    Valu2DJob<TC> g[kBandBoxes];
    int start[kBandBoxes + 1];  // first workgroup of each box
    TC w[K];
};

template <typename TS, typename TC, int SHAPE, int R, int T>
__global__ __launch_bounds__(64 * kValu2DWaves) void valu2d_band_kernel(
    Valu2DBandArgs<TC, Valu2DCfg<TS, TC, SHAPE, R, T, 1>::K> a)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, 1>;
    static_assert(!Cfg::WPTR, "weights in registers");
    const int wg = blockIdx.x;
    int j = 0;
    while (j + 1 < kBandBoxes && a.start[j + 1] <= wg) ++j;
    const Valu2DJob<TC> g = a.g[j];
    const int item = valu2d_item(wg - a.start[j]);
    if (item >= g.nbands * g.nsegs) return;
    const int seg = item / g.nbands, band = item - seg * g.nbands;
    TC wk[Cfg::K];
    load_weights<TC, Cfg::K>(wk, a.w);
    valu2d_tile<TS, TC, SHAPE, R, T, 1>(g, wk, nullptr, band, seg, threadIdx.x & 63);
}

// The boxes ps[0..n) of one pass (same grid, weights and boundary).
template <typename TS, typename TC, int SHAPE, int R, int T>
hipError_t launch_valu2d_band(const PassArgs *ps, int n, hipStream_t stream)
{
    using Cfg = Valu2DCfg<TS, TC, SHAPE, R, T, 1>;
    if (n < 1 || n > kBandBoxes) return hipErrorInvalidValue;
    static const int occ = valu2d_occupancy(valu2d_band_kernel<TS, TC, SHAPE, R, T>);
    Valu2DPick pick;
    valu2d_try<TS, TC, SHAPE, R, T, 1>(ps, n, occ, ps[0].num_cu > 0 ? ps[0].num_cu : 256, &pick);
    Valu2DBandArgs<TC, Cfg::K> a;
    int total = 0;
    for (int j = 0; j < kBandBoxes; ++j) {
        const PassArgs &p = ps[j < n ? j : n - 1];
        a.start[j] = total;
        valu2d_geometry<TS, TC, SHAPE, R, T, 1>(p, p.tile_rows > 0 ? p.tile_rows : pick.BY, &a.g[j]);
        if (j < n) total += a.g[j].nwg;
    }
    a.start[kBandBoxes] = total;
    for (int k = 0; k < Cfg::K; ++k) a.w[weight_slot<Cfg, R>(k)] = (TC)ps[0].w[k];
    hipLaunchKernelGGL((valu2d_band_kernel<TS, TC, SHAPE, R, T>), dim3(total), dim3(64 * kValu2DWaves), 0, stream, a);
    return hipGetLastError();
}

// Kernel-fused matrix passes of T >= 2 need their band redone (r = 7 has none).
template <typename TS, typename TC, int SHAPE, int R, int T>
constexpr hipError_t (*valu2d_band_launcher())(const PassArgs *, int, hipStream_t)
{
    if constexpr (T >= 2 && R <= 3) return &launch_valu2d_band<TS, TC, SHAPE, R, T>;
    else return nullptr;
}

#define V2(TS, TC, DT, SH, R, T) \
    {STENCIL_PATH_VALU, DT, SH, 2, R, T, &launch_valu2d<TS, TC, SH, R, T>, \
     &launch_valu2d_batch<TS, TC, SH, R, T>, valu2d_band_launcher<TS, TC, SH, R, T>()}
// Variants that only redo the Dirichlet band of a matrix pass.
#define V2_BAND(TS, TC, DT, SH, R, T) \
    {STENCIL_PATH_VALU, DT, SH, 2, R, T, nullptr, nullptr, valu2d_band_launcher<TS, TC, SH, R, T>()}
#define V2_BAND_T(TS, TC, DT, SH, R) \
    V2_BAND(TS, TC, DT, SH, R, 1), V2_BAND(TS, TC, DT, SH, R, 2), V2_BAND(TS, TC, DT, SH, R, 3), V2_BAND(TS, TC, DT, SH, R, 4)
#define V2_BAND_R(TS, TC, DT, SH) \
    V2_BAND_T(TS, TC, DT, SH, 1), V2_BAND_T(TS, TC, DT, SH, 2), V2_BAND_T(TS, TC, DT, SH, 3)
#define V2_BAND_S(TS, TC, DT) V2_BAND_R(TS, TC, DT, STENCIL_STAR), V2_BAND_R(TS, TC, DT, STENCIL_BOX)
#define V2_T(TS, TC, DT, SH, R) \
    V2(TS, TC, DT, SH, R, 1), V2(TS, TC, DT, SH, R, 2), V2(TS, TC, DT, SH, R, 3), V2(TS, TC, DT, SH, R, 4)
#define V2_R(TS, TC, DT, SH) V2_T(TS, TC, DT, SH, 1), V2_T(TS, TC, DT, SH, 2), V2_T(TS, TC, DT, SH, 3)
#define V2_S(TS, TC, DT) V2_R(TS, TC, DT, STENCIL_STAR), V2_R(TS, TC, DT, STENCIL_BOX)

}  // namespace stl
