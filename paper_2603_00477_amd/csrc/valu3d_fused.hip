// VALU path, d = 3, T explicit steps fused per pass (temporal fusion, paper
// Sec. "CUDA Core Implementation with Temporal Fusion": the intermediate
// fields of the T steps stay on chip, so a pass moves one field in and one out
// while its arithmetic grows with T, Eq. 8).
//
// Work decomposition
//   A workgroup of NW waves streams a segment of z planes.  Its in-plane
//   layout is 64 columns x NW*WY rows: a wave owns WY whole rows, a lane one
//   column of them.  With one column per lane any row length, alignment and
//   boundary takes the same path (each lane's source column is wrapped or
//   clamped once per tile), and the x neighbours are the neighbouring lanes.
//   Columns carry a skirt of R*T per side (BX = 64 - 2RT outputs); rows one of
//   R*(T-1), because the R input rows above and below the layout are staged.
//
// Step pipeline
//   Stage 0 takes input plane k (prefetched one plane ahead into registers).
//   Stage s = 1..T consumes the plane stage s-1 produced one iteration
//   earlier: the wave's own rows are still in its registers, the R rows above
//   and below come from the neighbouring waves through LDS, and the column
//   neighbours by whole-wave DPP rotates or, for the XL farthest columns of a
//   star, from the wave's own rows in LDS.  It scatters the plane into 2R+1
//   rotating accumulator planes (input plane z adds w[c][.][.] to output plane
//   z-c; contributions arrive with z, then rows, then columns ascending) and
//   emits the completed plane to the next stage or, for stage T, to HBM.  One
//   barrier per plane, fields double-buffered.
//
// What bounds it: vector issue.  Keeping a wave's own rows in registers leaves
// 2R row reads and at most WY row writes of LDS per plane and stage, where
// reading the whole (WY+2R) x (W+2R) window from LDS had made LDS the limit.
// 512^3 Dirichlet, us a pass, window-from-LDS kernel -> this one:
//   float32  Star-3D1R T2 299 -> 283     float64  Star-3D2R T2 607 -> 531
//            Star-3D2R T2 329 -> 321              Star-3D2R T3 863 -> 756
//            Star-3D2R T3 433 -> 398              Star-3D3R T2 833 -> 751
//            Star-3D3R T2 492 -> 417              Box-3D1R  T2 673 -> 587
//            Box-3D1R  T2 429 -> 355              Box-3D1R  T3 1009 -> 812
//            Box-3D1R  T3 570 -> 513
// and 97^3 float32 Star-3D1R T2 149 -> 7.8 us a pass: small grids need narrow
// tiles and short segments to reach every CU (see rows3d_pick).  Counters at
// 512^3 periodic: float32 and the float64 boxes issue vector instructions in
// 66-101 % of the cycles; the float64 Star-3D2R passes in 46-59 %, since their
// rows leave registers for 1.8 waves a SIMD.  LDS is busy in 4-46 %, without
// bank conflicts.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "internal.h"
#include "valu_common.h"

namespace stl {
namespace {

constexpr int kRowsMaxWaves = 8;
constexpr int kRowsMinWaves = 4;

// Geometry of one pass of one grid: output box, tiling and boundary.
template <typename TC, int K>
struct Rows3DArgs {
    const void *src;
    void *dst;
    int n0, n1, n2;
    int oz0, oz1, oy0, oy1, ox0, ox1;
    int BZ, BY, nty, ntx, nzs, ntiles;
    int periodic;
    TC h;
    TC w[K];
};

template <typename TC, int SHAPE, int R, int T, int WY, int XL>
struct Rows3DCfg {
    static constexpr int K = SHAPE == STENCIL_BOX ? (2 * R + 1) * (2 * R + 1) * (2 * R + 1) : 6 * R + 1;
    static constexpr int Q = 2 * R + 1;
    static constexpr int SK = R * (T - 1);      // rows of the exact margin, per side
    static constexpr int BX = 64 - 2 * R * T;   // output columns of a tile
    // planes prefetched (one-step passes move a plane per little arithmetic:
    // Box-3D1R float64 512^3 556 -> 447 us, Star-3D1R float32 267 -> 237 us
    // with two) and planes per unrolled loop body
    static constexpr int PF = T == 1 ? 2 : 1;
    static constexpr int U = Q * PF;
    static constexpr int NH = (2 * R + kRowsMinWaves - 1) / kRowsMinWaves;  // staged halo rows per wave
    // rows a wave keeps in LDS: all of them where columns are read back from
    // there, else the R first and R last ones its neighbours read
    static constexpr int SR = XL > 0 ? WY : 2 * R;
    static constexpr int SLOT = SR * 64;
    static_assert(WY >= R, "a wave's halo rows come from its direct neighbours");
    static_assert(BX > 0, "tile narrower than its skirt");
    static_assert(kRowsMinWaves * WY > 2 * SK, "layout lower than its margin");
    // per field: R halo rows, the waves' rows, R halo rows
    static constexpr int field(int nw) { return nw * SLOT + 2 * R * 64; }
    static constexpr int lds_bytes(int nw) { return 2 * T * field(nw) * (int)sizeof(TC); }
    static_assert(lds_bytes(kRowsMaxWaves) <= 160 * 1024, "fields exceed LDS");
};

// Value of the previous / next lane of the wave (whole-wave DPP rotate by one
// lane; the wrapped value at the wave's ends lies in the column skirt).  The
// destination's old value is left undefined: every lane is written, and a
// defined one costs a move per rotate.
template <bool PREV>
__device__ __forceinline__ int lane_rot(int v)
{
    return __builtin_amdgcn_mov_dpp(v, PREV ? 0x13C : 0x134, 0xF, 0xF, true);
}
template <bool PREV>
__device__ __forceinline__ float lane_rot(float v)
{
    return __int_as_float(lane_rot<PREV>(__float_as_int(v)));
}
template <bool PREV>
__device__ __forceinline__ double lane_rot(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = lane_rot<PREV>((int)(b & 0xffffffffLL)), hi = lane_rot<PREV>((int)(b >> 32));
    return __longlong_as_double(((long long)(unsigned)lo) | ((long long)hi << 32));
}

template <int R>
__device__ __forceinline__ constexpr int star3r_index(int axis, int off)
{
    return 1 + axis * 2 * R + (off < 0 ? off + R : off + R - 1);
}

// One tile (in-plane tile x plane segment) of one pass, run by the whole
// workgroup; `lds` holds the double-buffered rows of T fields.
template <typename TC, int SHAPE, int R, int T, int WY, int XL, int K>
__device__ __forceinline__ void rows3d_tile(const Rows3DArgs<TC, K> &a, const TC (&wk)[K], const int tile, TC *lds)
{
    using Cfg = Rows3DCfg<TC, SHAPE, R, T, WY, XL>;
    constexpr int Q = Cfg::Q, SK = Cfg::SK, NH = Cfg::NH, SLOT = Cfg::SLOT, PF = Cfg::PF, U = Cfg::U;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;

    const int tzs = tile / (a.nty * a.ntx);
    const int rem = tile - tzs * (a.nty * a.ntx);
    const int tyi = rem / a.ntx, txi = rem - tyi * a.ntx;
    const int z0 = a.oz0 + tzs * a.BZ, z1 = min(z0 + a.BZ, a.oz1);
    const int y0 = a.oy0 + tyi * a.BY, ye = min(y0 + a.BY, a.oy1);
    const int x0 = a.ox0 + txi * Cfg::BX, xe = min(x0 + Cfg::BX, a.ox1);
    const int n0 = a.n0, n1 = a.n1, n2 = a.n2;
    const bool periodic = a.periodic != 0;
    const TC h = a.h;
    const int64_t pitch = (int64_t)n1 * n2;

    // columns: this lane's source (wrapped, or a valid dummy whose value is
    // replaced by h) and whether it stores
    const int x = x0 - R * T + lane;
    const bool col_in = periodic || (x >= 0 && x < n2);
    const bool col_store = x >= x0 && x < xe;
    const TC *srcl = static_cast<const TC *>(a.src) + (periodic ? wrap(x, n2) : min(max(x, 0), n2 - 1));
    TC *dstl = static_cast<TC *>(a.dst) + x;
    // rows of the wave, the same for all its lanes
    const int yw = y0 - SK + wv * WY;
    int64_t roff[WY];
    unsigned rin = 0;
#pragma unroll
    for (int i = 0; i < WY; ++i) {
        const int y = yw + i;
        if (periodic || (y >= 0 && y < n1)) rin |= 1u << i;
        roff[i] = (int64_t)(periodic ? wrap(y, n1) : min(max(y, 0), n1 - 1)) * n2;
    }
    // input halo rows: row hr = wv + i nw of the 2R rows around the layout
    // (waves without one load a row of the halo again and do not write it)
    int64_t hoff[NH];
    int hlds[NH];
    bool hin[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) {
        const int hr = wv + i * nw;
        const int hc = hr < 2 * R ? hr : 0;
        const int y = hc < R ? y0 - SK - R + hc : y0 - SK + nw * WY + hc - R;
        hin[i] = periodic || (y >= 0 && y < n1);
        hoff[i] = (int64_t)(periodic ? wrap(y, n1) : min(max(y, 0), n1 - 1)) * n2;
        hlds[i] = hr >= 2 * R ? -1 : (hc < R ? hc * 64 : nw * SLOT + hc * 64) + lane;
    }
    const int BZe = z1 - z0, KIN = BZe + 2 * R * T, KTOT = KIN + T;
    const int zbase = z0 - R * T;
    const int FL = Cfg::field(nw);
    // the wave's first row in a field; the rows above it and below its last
    // one are the neighbours' (or the halo)
    const int own0 = R * 64 + wv * SLOT + lane;
    const int up0 = own0 - R * 64, dn0 = own0 + SLOT;

    TC acc[T][Q][WY], own[T][WY], ring[PF][WY], hring[PF][NH];
#pragma unroll
    for (int s = 0; s < T; ++s)
#pragma unroll
        for (int i = 0; i < WY; ++i) {
            own[s][i] = TC(0);
#pragma unroll
            for (int q = 0; q < Q; ++q) acc[s][q][i] = TC(0);
        }
    int zl = periodic ? wrap(zbase, n0) : 0;  // periodic: source plane of the next load
    auto load_plane = [&](int k, TC (&r)[WY], TC (&hr)[NH]) {
        const int z = periodic ? zl : min(max(zbase + k, 0), n0 - 1);
        const int64_t zoff = (int64_t)z * pitch;
        // opaque scalar offsets: the rows' addresses are not worth the vector
        // registers that hoisting them out of the loop takes (Box-3D1R
        // float32 T = 2: 117 instead of 80)
        auto row_at = [&](int64_t off) {
            off += zoff;
            asm volatile("" : "+s"(off));
            return srcl[off];
        };
#pragma unroll
        for (int i = 0; i < WY; ++i) r[i] = row_at(roff[i]);
#pragma unroll
        for (int i = 0; i < NH; ++i) hr[i] = row_at(hoff[i]);
        zl = zl + 1 == n0 ? 0 : zl + 1;
    };
    // the wave's rows of a field, to where its neighbours (and itself) read them
    auto put_row = [&](TC *wr, int i, TC v) {
        if constexpr (XL > 0) {
            wr[i * 64] = v;
        } else {
            if (i < R) wr[i * 64] = v;
            if (i >= WY - R) wr[(i - WY + 2 * R) * 64] = v;
        }
    };
#pragma unroll
    for (int k = 0; k < PF; ++k) load_plane(k, ring[k], hring[k]);

    for (int kb = 0; kb < KTOT; kb += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = kb + u;
            if (k >= KTOT) break;
            const int par = (U % 2 ? k : u) & 1;
            // stages from T down to 1: each has used its predecessor's rows of
            // the previous iteration before that one replaces them
#pragma unroll
            for (int s = T; s >= 1; --s) {
                const bool active = k >= s + 2 * R * (s - 1) && k < KIN + s;
                if (!active) continue;
                const TC *rd = lds + (2 * (s - 1) + (par ^ 1)) * FL;
                TC up[R], dn[R];
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    up[m] = rd[up0 + m * 64];
                    dn[m] = rd[dn0 + m * 64];
                }
#pragma unroll
                for (int wi = 0; wi < WY + 2 * R; ++wi) {
                    const bool mid = wi >= R && wi < R + WY;  // a row of this wave
                    TC row[Q];  // columns lane - R .. lane + R
                    row[R] = wi < R ? up[wi] : (mid ? own[s - 1][wi - R] : dn[wi - R - WY]);
                    if (SHAPE == STENCIL_BOX || mid) {
#pragma unroll
                        for (int m = 1; m <= R; ++m) {
                            if (m > R - XL) {
                                row[R - m] = rd[own0 + (wi - R) * 64 - m];
                                row[R + m] = rd[own0 + (wi - R) * 64 + m];
                            } else {
                                row[R - m] = lane_rot<true>(row[R - m + 1]);
                                row[R + m] = lane_rot<false>(row[R + m - 1]);
                            }
                        }
                    }
#pragma unroll
                    for (int c = -R; c <= R; ++c) {
                        const int q = ((u - c + R) % Q + Q) % Q;
#pragma unroll
                        for (int i = 0; i < WY; ++i) {
                            const int ao = wi - i - R;
                            if (ao < -R || ao > R) continue;
                            TC &o = acc[s - 1][q][i];
                            // the first contribution (c = -R, first row and
                            // column) starts the sum, from zero: a product alone
                            // would keep the sign of a zero
                            if constexpr (SHAPE == STENCIL_BOX) {
#pragma unroll
                                for (int bo = -R; bo <= R; ++bo) {
                                    const TC wv_ = wk[((c + R) * Q + (ao + R)) * Q + (bo + R)];
                                    o = fma_c(wv_, row[bo + R], c == -R && ao == -R && bo == -R ? TC(0) : o);
                                }
                            } else if (c != 0) {  // z arm: own column only
                                if (ao != 0) continue;
                                const TC wv_ = wk[star3r_index<R>(0, c)];
                                o = fma_c(wv_, row[R], c == -R ? TC(0) : o);
                            } else if (ao != 0) {  // y arm
                                o = fma_c(wk[star3r_index<R>(1, ao)], row[R], o);
                            } else {  // x arm with the centre
#pragma unroll
                                for (int bo = -R; bo <= R; ++bo)
                                    o = fma_c(bo == 0 ? wk[0] : wk[star3r_index<R>(2, bo)], row[bo + R], o);
                            }
                        }
                    }
                }
                const int zo = zbase + k - s * (1 + R);
                const int qc = u % Q;  // accumulator plane completed now
                if (s < T) {
                    const bool zin = periodic || (zo >= 0 && zo < n0);
                    TC *wr = lds + (2 * s + par) * FL + own0;
#pragma unroll
                    for (int i = 0; i < WY; ++i) {
                        const TC v = (zin && ((rin >> i) & 1u) && col_in) ? acc[s - 1][qc][i] : h;
                        own[s < T ? s : 0][i] = v;
                        put_row(wr, i, v);
                    }
                } else if (zo >= z0 && zo < z1) {
                    int64_t off = (int64_t)zo * pitch + (int64_t)yw * n2;
                    asm volatile("" : "+s"(off));
                    TC *pl = dstl + off;
#pragma unroll
                    for (int i = 0; i < WY; ++i) {
                        const int y = yw + i;
                        if (y >= y0 && y < ye && col_store) pl[(int64_t)i * n2] = acc[s - 1][qc][i];
                    }
                }
            }
            // stage 0: input plane k and its halo rows become field 0
            {
                const bool zin = periodic || (zbase + k >= 0 && zbase + k < n0);
                TC *wr = lds + par * FL;
#pragma unroll
                for (int i = 0; i < WY; ++i) {
                    const TC v = (zin && ((rin >> i) & 1u) && col_in) ? ring[u % PF][i] : h;
                    own[0][i] = v;
                    put_row(wr + own0, i, v);
                }
#pragma unroll
                for (int i = 0; i < NH; ++i) {
                    const TC v = (zin && hin[i] && col_in) ? hring[u % PF][i] : h;
                    if (hlds[i] >= 0) wr[hlds[i]] = v;
                }
                // keep the refill of the ring behind the reads that drain it
                __builtin_amdgcn_sched_barrier(0);
                if (k + PF < KIN) load_plane(k + PF, ring[u % PF], hring[u % PF]);
            }
            __syncthreads();
        }
    }
}

// Float32 weights are pinned in vector registers (float32 FMAs with a scalar
// operand issue slower on gfx950).
template <typename TC, int K>
__device__ __forceinline__ void rows3d_weights(TC (&wk)[K], const TC *w)
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        wk[k] = w[k];
        if constexpr (sizeof(TC) == 4) asm volatile("" : "+v"(wk[k]));
    }
}

extern __shared__ __attribute__((aligned(16))) unsigned char rows3d_lds[];

template <typename TC, int SHAPE, int R, int T, int WY, int XL, int MINW>
__global__ __launch_bounds__(64 * kRowsMaxWaves) __attribute__((amdgpu_waves_per_eu(MINW))) void fused3d_kernel(
    Rows3DArgs<TC, Rows3DCfg<TC, SHAPE, R, T, WY, XL>::K> a)
{
    using Cfg = Rows3DCfg<TC, SHAPE, R, T, WY, XL>;
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    if (tile >= a.ntiles) return;
    TC wk[Cfg::K];
    rows3d_weights<TC, Cfg::K>(wk, a.w);
    rows3d_tile<TC, SHAPE, R, T, WY, XL, Cfg::K>(a, wk, tile, reinterpret_cast<TC *>(rows3d_lds));
}

// Persistent batched launch: the workgroups walk one list of tiles spanning
// every job of the batch; workgroup b takes items b + i*gridDim.  tile_start[j]
// is the first item of job j (tile_start[njobs] = total).  The tile body ends
// with a barrier, so the LDS rows are free when the next item starts.
template <typename TC, int SHAPE, int R, int T, int WY, int XL, int MINW>
__global__ __launch_bounds__(64 * kRowsMaxWaves) __attribute__((amdgpu_waves_per_eu(MINW))) void fused3d_batch_kernel(
    const Rows3DArgs<TC, Rows3DCfg<TC, SHAPE, R, T, WY, XL>::K> *__restrict__ jobs,
    const int *__restrict__ tile_start, int njobs)
{
    using Cfg = Rows3DCfg<TC, SHAPE, R, T, WY, XL>;
    const int total = tile_start[njobs];
    int j = 0;
    for (int item = xcd_remap(blockIdx.x, gridDim.x); item < total; item += gridDim.x) {
        while (j + 1 < njobs && tile_start[j + 1] <= item) ++j;
        const Rows3DArgs<TC, Cfg::K> a = jobs[j];
        TC wk[Cfg::K];
        rows3d_weights<TC, Cfg::K>(wk, jobs[j].w);
        rows3d_tile<TC, SHAPE, R, T, WY, XL, Cfg::K>(a, wk, item - tile_start[j], reinterpret_cast<TC *>(rows3d_lds));
    }
}

// Rows per wave, farthest columns read from LDS, and waves per SIMD the
// registers are held to.  Measured on 512^3 over WY = 4..8, XL = 0..2 and 4 or
// 8 waves: as many rows as two resident 8-wave workgroups (128 registers;
// float64 stars with r >= 2: one, 256) have room for, since every row of the
// margin is recomputed by each tile; XL >= 1 gains 2-11 % where rotates are
// the larger share (Star-3D2R float32 T = 3 1019 -> 1131 GSt/s) and loses 3 %
// on Star-3D2R float64 T = 3 and Star-3D1R, whose one rotate per side is
// cheap.  One-step passes have no margin and take four rows.
template <typename TC, int SHAPE, int R, int T>
struct Rows3DShape {
    static constexpr bool F64 = sizeof(TC) == 8, BOX = SHAPE == STENCIL_BOX;
    static constexpr int WY = T == 1 || BOX || R == 1 ? (!F64 && T == 3 ? 6 : 4) : (F64 && R == 2 && T == 2 ? 6 : 5);
    static constexpr int XL = BOX || R == 1               ? 0
                              : T == 1 || (F64 && T == 2) ? 1
                              : F64                       ? 0
                                                          : (R == 2 && T == 3 ? 1 : 2);
    static constexpr int MINW = F64 && (R == 3 || (R == 2 && T > 1)) ? 1 : 4;
};

// One in-plane box of a launch: planes, rows and columns to write.
struct Box3 {
    int d0, d1, d2;
};

struct Rows3DPick {
    int nw, BZ;
};

// Waves per workgroup (4 or 8) and planes per segment of a launch over n
// boxes, by an estimate in cycles of a launch's time: the root of the squares
// of its issue time and its bytes' time.
//   issue: a workgroup takes BZ + 2RT + T plane iterations (the lead-in ones,
//     where later stages idle, count 0.2) and the worth of 3.7 more to start;
//     one costs a latency (barrier, LDS, the next plane's loads) and the
//     arithmetic of the waves that share a SIMD; times the rounds over the
//     resident workgroups.
//   bytes: one read and one write per point, and a fifth of what the tiles'
//     margins and lead-in planes read again (caches hold the rest), at 1600 a
//     cycle.
// Lengths from one plane to 512 are tried, whatever the height (a tall grid
// once fell through to a single segment: 6000 x 32^2 float32 Star-3D1R 3284 us
// instead of 48).  Small grids come out with segments of a few planes that put
// work on every CU (48^3 float32 Star-3D1R T = 2: 1 plane 5.4 us, 4 planes 7.9;
// 97^3: 3 planes 9.7, 33 planes 25), large ones with segments that amortise
// the lead-in planes in whole rounds (512^3 Star-3D2R float64 T = 3: 171 planes
// 738 us, 128 871).  r = 1 and one-step passes are near the memory bound at
// large sizes and gain from neighbouring tiles running close in time: at most
// 16 R T planes (512^3 Star-3D1R float64 T = 2: 171 planes 549 us, 32 502).
// Fitted to 11 variants in float32 and float64 on 62 grids (32^3..512^3, flat,
// tall, and at random): the choice is 1 % behind the best of all measured
// lengths on average, 24 % at most (float64 r = 3 one-step passes of
// 128 x 640^2).
template <typename Cfg, typename TC, int SHAPE, int R, int T, int WY>
Rows3DPick rows3d_pick(const Box3 *boxes, int n, int fixed_bz, int cus, const int (&occ)[2])
{
    constexpr bool F64 = sizeof(TC) == 8;
    const double wave = T * WY * ((F64 ? 5.5 : 2.0) * Cfg::K + 3.2 * (2 * R * (sizeof(TC) / 4) + 16));
    const double latency = (F64 ? 950.0 : 600.0) + 400.0 * T;
    static const int kPlanes[] = {1,  2,  3,  4,  5,  6,  7,  8,  9,  10, 11, 12, 13, 14,  16,  18,  20, 22,
                                  24, 28, 32, 37, 43, 48, 52, 57, 64, 74, 86, 103, 128, 171, 256, 512};
    int dmax = 1;
    double points = 0;
    for (int i = 0; i < n; ++i) {
        dmax = std::max(dmax, boxes[i].d0);
        points += (double)boxes[i].d0 * boxes[i].d1 * boxes[i].d2;
    }
    Rows3DPick best{kRowsMaxWaves, dmax};
    double best_cost = -1.0;
    for (int v = 0; v < 2; ++v) {
        const int nw = v ? kRowsMaxWaves : kRowsMinWaves, BY = nw * WY - 2 * Cfg::SK;
        const int slots = cus * occ[v];
        int last = 0;
        for (int most : kPlanes) {
            if ((R == 1 || T == 1) && most > 16 * R * T) break;
            const int segs = (dmax + most - 1) / most;
            const int BZ = fixed_bz > 0 ? fixed_bz : (dmax + segs - 1) / segs;
            if (BZ == last) continue;
            last = BZ;
            double items = 0;
            for (int i = 0; i < n; ++i)
                items += (double)((boxes[i].d0 + BZ - 1) / BZ) * ((boxes[i].d1 + BY - 1) / BY) *
                         ((boxes[i].d2 + Cfg::BX - 1) / Cfg::BX);
            const double full = (double)(int64_t)(items / slots);
            const double rest = items - full * slots;
            auto plane = [&](double resident) {  // cycles of a plane iteration
                const double perSimd = (double)(int64_t)((resident * nw + 3) / 4);
                return latency + wave * perSimd;
            };
            double rounds = full * plane(occ[v]);
            if (rest > 0) rounds += plane((double)(int64_t)((rest + cus - 1) / cus));
            const int BZe = std::min(BZ, dmax);
            const double issue = (BZe + 0.2 * (2 * R * T + T) + 3.7) * rounds;
            const double read = items * (BZe + 2 * R * T) * (nw * WY + 2 * R) * 64;
            const double bytes = sizeof(TC) * (2 * points + 0.2 * std::max(read - points, 0.0)) / 1600.0;
            const double cost = issue * issue + bytes * bytes;
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = {nw, BZ};
            }
        }
    }
    return best;
}

inline Box3 box_of(const PassArgs &p)
{
    return {p.region_hi[0] - p.region_lo[0], p.region_hi[1] - p.region_lo[1], p.region_hi[2] - p.region_lo[2]};
}

// Fill the arguments of one pass; returns false when there is nothing to do
// (err then says whether the pass is invalid).
template <typename Cfg, typename TC, int WY>
bool rows3d_args(const PassArgs &p, Rows3DPick pick, Rows3DArgs<TC, Cfg::K> *out, hipError_t *err)
{
    *err = hipSuccess;
    Rows3DArgs<TC, Cfg::K> &a = *out;
    a.src = p.src;
    a.dst = p.dst;
    a.n0 = (int)p.dims[0];
    a.n1 = (int)p.dims[1];
    a.n2 = (int)p.dims[2];
    a.oz0 = p.region_lo[0];
    a.oz1 = p.region_hi[0];
    a.oy0 = p.region_lo[1];
    a.oy1 = p.region_hi[1];
    a.ox0 = p.region_lo[2];
    a.ox1 = p.region_hi[2];
    a.periodic = p.boundary == STENCIL_PERIODIC;
    a.h = (TC)p.halo;
    for (int k = 0; k < Cfg::K; ++k) a.w[k] = (TC)p.w[k];
    const Box3 b = box_of(p);
    if (b.d0 <= 0 || b.d1 <= 0 || b.d2 <= 0) return false;
    a.BY = pick.nw * WY - 2 * Cfg::SK;
    a.nty = (b.d1 + a.BY - 1) / a.BY;
    a.ntx = (b.d2 + Cfg::BX - 1) / Cfg::BX;
    const int64_t inplane = (int64_t)a.nty * a.ntx, most = 1LL << 30;
    if (inplane > most) {
        *err = hipErrorInvalidValue;
        return false;
    }
    // segments of equal length, no more of them than tile ids allow
    int64_t segs = (b.d0 + pick.BZ - 1) / pick.BZ;
    if (p.tile_rows > 0) {
        a.BZ = p.tile_rows;
        if (segs * inplane > most) {
            *err = hipErrorInvalidValue;
            return false;
        }
    } else {
        segs = std::min<int64_t>(segs, most / inplane);
        a.BZ = (int)((b.d0 + segs - 1) / segs);
    }
    a.nzs = (b.d0 + a.BZ - 1) / a.BZ;
    a.ntiles = (int)(a.nzs * inplane);
    return true;
}

// resident workgroups per CU with 4 and with 8 waves
template <typename Cfg, typename K>
struct Rows3DOcc {
    int occ[2];
    explicit Rows3DOcc(K kernel)
    {
        for (int v = 0; v < 2; ++v) {
            const int nw = v ? kRowsMaxWaves : kRowsMinWaves;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ[v], kernel, 64 * nw, Cfg::lds_bytes(nw)) !=
                    hipSuccess || occ[v] < 1)
                occ[v] = 1;
        }
    }
};

template <typename Cfg, typename K>
hipError_t rows3d_allow_lds(K kernel, int nw)
{
    if (Cfg::lds_bytes(nw) <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               Cfg::lds_bytes(nw));
}

template <typename TC, int SHAPE, int R, int T>
hipError_t launch_fused3d(const PassArgs &p, hipStream_t stream)
{
    using S = Rows3DShape<TC, SHAPE, R, T>;
    using Cfg = Rows3DCfg<TC, SHAPE, R, T, S::WY, S::XL>;
    const auto kernel = fused3d_kernel<TC, SHAPE, R, T, S::WY, S::XL, S::MINW>;
    static const Rows3DOcc<Cfg, decltype(kernel)> occ(kernel);
    const Box3 b = box_of(p);
    const Rows3DPick pick = rows3d_pick<Cfg, TC, SHAPE, R, T, S::WY>(&b, 1, p.tile_rows, p.num_cu > 0 ? p.num_cu : 256,
                                                                     occ.occ);
    Rows3DArgs<TC, Cfg::K> a;
    hipError_t err;
    if (!rows3d_args<Cfg, TC, S::WY>(p, pick, &a, &err)) return err;
    if ((int64_t)a.ntiles * 64 * pick.nw > UINT32_MAX) {
        // a launch takes less than 2^32 threads (one column a lane: some 1.5e10
        // points in a plane or two): the halves of the box after each other
        const int ax = b.d1 >= b.d2 ? 1 : 2, mid = p.region_lo[ax] + (ax == 1 ? b.d1 : b.d2) / 2;
        PassArgs lower = p, upper = p;
        lower.region_hi[ax] = upper.region_lo[ax] = mid;
        err = launch_fused3d<TC, SHAPE, R, T>(lower, stream);
        return err == hipSuccess ? launch_fused3d<TC, SHAPE, R, T>(upper, stream) : err;
    }
    err = rows3d_allow_lds<Cfg>(kernel, pick.nw);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kernel, dim3(a.ntiles), dim3(64 * pick.nw), Cfg::lds_bytes(pick.nw), stream, a);
    return hipGetLastError();
}

template <typename TC, int SHAPE, int R, int T>
hipError_t launch_fused3d_batch(const PassArgs *ps, int n, BatchStaging *stage, hipStream_t stream)
{
    using S = Rows3DShape<TC, SHAPE, R, T>;
    using Cfg = Rows3DCfg<TC, SHAPE, R, T, S::WY, S::XL>;
    using Args = Rows3DArgs<TC, Cfg::K>;
    const auto kernel = fused3d_batch_kernel<TC, SHAPE, R, T, S::WY, S::XL, S::MINW>;
    static const Rows3DOcc<Cfg, decltype(kernel)> occ(kernel);
    const int cus = ps[0].num_cu > 0 ? ps[0].num_cu : 256;
    std::vector<Box3> boxes;
    for (int i = 0; i < n; ++i) {
        const Box3 b = box_of(ps[i]);
        if (b.d0 > 0 && b.d1 > 0 && b.d2 > 0) boxes.push_back(b);
    }
    if (boxes.empty()) return hipSuccess;
    const Rows3DPick pick =
        rows3d_pick<Cfg, TC, SHAPE, R, T, S::WY>(boxes.data(), (int)boxes.size(), 0, cus, occ.occ);
    std::vector<Args> jobs;
    std::vector<int> start(1, 0);
    jobs.reserve(n);
    for (int i = 0; i < n; ++i) {
        Args a;
        hipError_t err;
        if (!rows3d_args<Cfg, TC, S::WY>(ps[i], {pick.nw, ps[i].tile_rows > 0 ? ps[i].tile_rows : pick.BZ}, &a, &err)) {
            if (err != hipSuccess) return err;
            continue;
        }
        if ((int64_t)start.back() + a.ntiles > (1LL << 30)) return hipErrorInvalidValue;
        jobs.push_back(a);
        start.push_back(start.back() + a.ntiles);
    }
    void *djobs = nullptr, *dstart = nullptr;
    hipError_t e = stage_job_table(stage, jobs.data(), jobs.size() * sizeof(Args), start, &djobs, &dstart,
                                   stream);
    if (e == hipSuccess) e = rows3d_allow_lds<Cfg>(kernel, pick.nw);
    if (e != hipSuccess) return e;
    const int total = start.back(), slots = cus * occ.occ[pick.nw == kRowsMaxWaves];
    hipLaunchKernelGGL(kernel, dim3(total < slots ? total : slots), dim3(64 * pick.nw), Cfg::lds_bytes(pick.nw), stream,
                       static_cast<const Args *>(djobs), static_cast<const int *>(dstart), (int)jobs.size());
    return hipGetLastError();
}

// One-step passes.  Large grids whose rows are whole aligned vectors go to the
// 16-byte-load kernel of valu3d.hip, which moves HBM traffic 3-10 % faster
// (512^3: float32 Star-3D1R 230 vs 237 us, float64 Box-3D1R 411 vs 447; 320^3
// float64 Star-3D1R 114 vs 125); below 384 MB in and out, where the last-level
// cache (256 MB) holds much of a pass, and for other row lengths the narrow
// tiles above win (256^3 float32 Star-3D1R 33 vs 27 us, 333^3 120 vs 72, 97^3
// 40 vs 7.5).  Float64 Star-3D3R is bound by its arithmetic and wins at every
// size (512^3 524 vs 517 us, 97^3 48 vs 12.7).
template <typename TC, int R>
bool one_step_streams(const PassArgs &p)
{
    if (sizeof(TC) == 8 && R == 3) return false;
    const int64_t row = p.dims[2] * (int)sizeof(TC), bytes = 2 * p.dims[0] * p.dims[1] * row;
    bool whole = true;
    for (int i = 0; i < 3; ++i) whole = whole && p.region_lo[i] == 0 && p.region_hi[i] == p.dims[i];
    return whole && bytes >= (384LL << 20) && row % 16 == 0 && ((uintptr_t)p.src | (uintptr_t)p.dst) % 16 == 0;
}

template <typename TC, int DT, int SHAPE, int R>
hipError_t launch_one_step3d(const PassArgs &p, hipStream_t stream)
{
    if (one_step_streams<TC, R>(p)) return valu3d_stream_kernel(DT, SHAPE, R)->launch(p, stream);
    return launch_fused3d<TC, SHAPE, R, 1>(p, stream);
}

template <typename TC, int DT, int SHAPE, int R>
hipError_t launch_one_step3d_batch(const PassArgs *ps, int n, BatchStaging *stage, hipStream_t stream)
{
    std::vector<PassArgs> large, other;
    for (int i = 0; i < n; ++i) (one_step_streams<TC, R>(ps[i]) ? large : other).push_back(ps[i]);
    hipError_t e = hipSuccess;
    if (!large.empty())
        e = valu3d_stream_kernel(DT, SHAPE, R)->launch_batch(large.data(), (int)large.size(), stage, stream);
    if (e == hipSuccess && !other.empty())
        e = launch_fused3d_batch<TC, SHAPE, R, 1>(other.data(), (int)other.size(), stage, stream);
    return e;
}

#define F3_1(TC, DT, SH, R) \
    {STENCIL_PATH_VALU, DT, SH, 3, R, 1, &launch_one_step3d<TC, DT, SH, R>, &launch_one_step3d_batch<TC, DT, SH, R>}
#define F3(TC, DT, SH, R, T) \
    {STENCIL_PATH_VALU, DT, SH, 3, R, T, &launch_fused3d<TC, SH, R, T>, &launch_fused3d_batch<TC, SH, R, T>}
#define F3_S(TC, DT)                                                                                  \
    F3(TC, DT, STENCIL_STAR, 1, 2), F3(TC, DT, STENCIL_STAR, 1, 3), F3(TC, DT, STENCIL_STAR, 2, 2),   \
        F3(TC, DT, STENCIL_STAR, 2, 3), F3(TC, DT, STENCIL_STAR, 3, 2), F3(TC, DT, STENCIL_BOX, 1, 2), \
        F3(TC, DT, STENCIL_BOX, 1, 3), F3_1(TC, DT, STENCIL_STAR, 1), F3_1(TC, DT, STENCIL_STAR, 2),  \
        F3_1(TC, DT, STENCIL_STAR, 3), F3_1(TC, DT, STENCIL_BOX, 1)

}  // namespace

const std::vector<KernelEntry> &valu3d_fused_kernels()
{
    static const std::vector<KernelEntry> table = {
        F3_S(double, STENCIL_F64),
        F3_S(float, STENCIL_F32),
    };
    return table;
}

}  // namespace stl
