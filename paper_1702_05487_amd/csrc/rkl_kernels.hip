// rkl_kernels.hip -- single-grid kernels of librkl for gfx950: the
// temperature min/max reduction, the finalize step that turns it into
// dt_par, the stage count s and the stage scale (Sec. 3.1 Eq. dt_exp,
// Sec. 3.3 Eq. RKL-s, Sec. 4.1 rounding), and the stencil/stage kernels that
// wrap run_tile (rkl_tile.h).
#include <algorithm>
#include <cmath>

#include "rkl_stage.h"

namespace rkl {

// ------------------------------------------------------------ variants ----
// (bx, by) are compile-time tile shapes; bz is the z-chunk length per block;
// fuse is the number of stages per launch (F = 2..4: rkl_fused.hip, where
// (bx, by) is the region of a workgroup and (bx-2(F-1), by-2(F-1)) its
// output tile).  Variant 0 is the library's choice by the grid, with chunks of
// at most 64 planes; so are the one-stage launches of the fused variants.
static const Variant kVariants[] = {
    {32, 8, 64, 1},        {32, 8, 64, 1, true},  {64, 4, 32, 1, true}, {64, 4, 64, 1, true}, {16, 16, 32, 1, true},
    {16, 16, 64, 1, true}, {32, 8, 16, 1, true},  {64, 4, 16, 1, true},
    {16, 16, 32, 2},       {16, 16, 64, 2},       {32, 8, 32, 2},       {32, 8, 64, 2},
    {16, 16, 32, 3},       {16, 16, 64, 3},       {16, 16, 32, 4},      {16, 16, 64, 4},
    {32, 8, 32, 1, true},
};
int variant_count() { return (int)(sizeof(kVariants) / sizeof(kVariants[0])); }
Variant variant_get(int v) { return kVariants[v]; }

// ----------------------------------------------------------- reduction ----
// per-block maximum, minimum and a non-finite flag of T
__global__ __launch_bounds__(256) void reduce_minmax_kernel(const double* __restrict__ T, int64_t N,
                                                            double* __restrict__ part,
                                                            const int32_t* __restrict__ skip) {
    if (skip && *skip) return;   // uniform: the extrema are already there
    double mx = -INFINITY, mn = INFINITY, bad = 0.0;
    const int64_t step = (int64_t)gridDim.x * 256;
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (; i + 3 * step < N; i += 4 * step) {   // four loads in flight per lane
        const double v0 = T[i], v1 = T[i + step], v2 = T[i + 2 * step], v3 = T[i + 3 * step];
        mx = fmax(mx, fmax(fmax(v0, v1), fmax(v2, v3)));
        mn = fmin(mn, fmin(fmin(v0, v1), fmin(v2, v3)));
        bad = isfinite(v0) && isfinite(v1) && isfinite(v2) && isfinite(v3) ? bad : 1.0;
    }
    for (; i < N; i += step) {
        const double v = T[i];
        mx = fmax(mx, v);
        mn = fmin(mn, v);
        bad = isfinite(v) ? bad : 1.0;
    }
    for (int off = 32; off > 0; off >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, off));
        mn = fmin(mn, __shfl_xor(mn, off));
        bad = fmax(bad, __shfl_xor(bad, off));
    }
    __shared__ double sm[3][4];
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    if (l == 0) { sm[0][w] = mx; sm[1][w] = mn; sm[2][w] = bad; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 4; ++i) {
            mx = fmax(mx, sm[0][i]);
            mn = fmin(mn, sm[1][i]);
            bad = fmax(bad, sm[2][i]);
        }
        part[3 * blockIdx.x + 0] = mx;
        part[3 * blockIdx.x + 1] = mn;
        part[3 * blockIdx.x + 2] = bad;
    }
}

int reduce_blocks(int64_t N) {
    int64_t b = (N + 255) / 256;
    if (b > 1024) b = 1024;
    if (b < 1) b = 1;
    return (int)b;
}

hipError_t launch_reduce(const double* T, int64_t N, double* partials, int nblocks, hipStream_t st,
                         const int32_t* skip) {
    reduce_minmax_kernel<<<nblocks, 256, 0, st>>>(T, N, partials, skip);
    return hipGetLastError();
}

__global__ __launch_bounds__(1024) void finalize_kernel(GridConst g, StateSource q, GridState* st,
                                                        int32_t* ext_clear) {
    __shared__ double red[3][16];
    __shared__ GridState o;
    block_state(g, q, true, st, red, &o);
    if (ext_clear && threadIdx.x == 0) *ext_clear = 0;   // every lane has read it
}

hipError_t launch_finalize(const GridConst& gc, const StateSource& q, GridState* state, int32_t* ext_clear,
                           hipStream_t st) {
    finalize_kernel<<<1, q.field || q.ext_n > 1024 ? 1024 : 256, 0, st>>>(gc, q, state, ext_clear);
    return hipGetLastError();
}

// -------------------------------------------------------- stage kernels ----
// (instantiated in the rkl_stage_*.hip units)
template <typename R>
static hipError_t launch_prec(const StageLaunch& P, int nblocks, const Variant& v, bool lim, int sat,
                              hipStream_t st) {
    if (v.block) return launch_block<R>(P, nblocks, lim, sat, st);
    const int bx = v.bx, by = v.by;
    // grids with fixed axes: one runtime-shaped 16 x 16 kernel with the ghost loads
    if (P.t.fixed) return bx == 16 && by == 16 ? launch_fixed<R>(P, nblocks, lim, sat, st)
                                               : hipErrorInvalidValue;
    if (bx == 32 && by == 8) return launch_shape<R, 32, 8>(P, nblocks, lim, sat, st);
    if (bx == 64 && by == 4) return launch_shape<R, 64, 4>(P, nblocks, lim, sat, st);
    if (bx == 16 && by == 16) return launch_shape<R, 16, 16>(P, nblocks, lim, sat, st);
    return hipErrorInvalidValue;
}

// How a one-stage launch on a 3-D grid is split.
//
// Marched tiles (run_tile): a workgroup marches its z-chunk plane after plane,
// each plane a chain of one barrier, LDS exchanges and three face evaluations,
// so a launch takes as long as its longest march times the rounds of resident
// workgroups.  A chunk of bz planes costs bz + 2 plane iterations (the two
// before z0 fill the rings); an iteration takes chunk[k] microseconds with k
// workgroups on a CU.  Short chunks give a small grid enough workgroups for the
// 256 CUs, long ones keep the two extra iterations and the halo planes cheap.
// The last, partly filled round is priced half by its share of the slots and half
// as a round of its own: workgroups of different rounds overlap, but not fully.
// Two rounds and more of the classical flux, which loads more than it computes, end
// 0.15 of a march late, between one and two rounds a share of that (256^3, kappa0,
// chunks of 64 / 32 planes: FP64 241 / 227 us a stage, mixed 175 / 165; with T^2.5
// 259 / 259 and 170 / 170; 176^3 FP64, T^2.5, 26 / 16 planes: 99 / 96).
//
// Blocks of 16 x 4 x 4 cells (rkl_block.h) have no march; n of them take
// max(least, b0 + b1 n) microseconds.  The march's own time for the comparison is
// start + (bz + lead) x rounds with it[k] an iteration and `mix` of the last
// round as its own.  start to b1 are fits to 34 sizes from 8 x 8 x 512 to 2^22 cells,
// every chunk, with the kernels as they are now (rms 2 to 5 %; FP64 without
// saturation 9 %).  Beyond 2^22 cells the memory sets the time of both, and the
// march reads less of it.  FP64 with pow() marches at one wave per SIMD (its
// kernel takes 264 registers, the block kernel 127), so blocks stay faster there
// up to the largest grid measured (384^3).
//
// Measured, us a stage, best march (its chunk) / blocks; x: not taken:
//                     FP64, T^2.5, saturated  mixed, the same     FP64, T^1.7, upwind
//   24^3              x 7.5 (1)    5.8        x 6.6 (1)    5.4    x 11.1 (1)     7.8
//   64^3              x 11.2 (2)   9.4        x 9.2 (2)    7.6    x 22.5 (4)    14.9
//   88^3              19.2 (4)  x 19.1        13.5 (4)  x 13.7    x 56.3 (6)    34.7
//   112^3             x 36.0 (10) 32.6        x 23.0 (10) 21.9    x 107 (28)    60.5
//   128^3             42.5 (12) x 46.0        26.7 (12) x 29.9    x 124 (32)    90.2
//   150 x 127 x 101   43.2 (12) x 46.2        26.8 (12) x 30.6    x 128 (34)    90.3
//   65 x 65 x 300     x 50.7 (16) 34.4        x 30.0 (16) 24.0    x 154 (20)    68.9
//   512 x 512 x 1     13.7 (1)  x 22.8        11.2 (1)  x 15.8    35.7 (1)    x 43.7
//   512 x 512 x 4     x 26.0 (4)  24.2        x 19.5 (4)  17.0    x 80.7 (4)    44.6
//   192^3             126 (16)  x 159         75.1 (39) x 101     x 437 (39)     285
Variant fit_variant(int precision, Variant v, const GridConst& gc) {
    if (gc.fixed) {
        v.bx = v.by = 16;   // the tile shape of the ghost-loading kernel
        v.fuse = 1;
    }
    if (v.exact) return v;
    if (gc.fixed) v.bz = std::min(v.bz, 32);   // 256^3 mixed: 32 planes 222, 64 planes 254 us
    const bool f32 = precision == RKL_MIXED;
    const bool pow_law = gc.kmode == 2, sat = gc.saturation != 0;
    struct Price {
        int per_cu;   // workgroups on a CU, by registers and LDS
        double chunk[5];
        double start, lead, mix, it[4], least, b0, b1;
    };
    static const Price prices[] = {
        // FP64: classical, saturated (three_waves), pow()
        {2, {0, 1.3, 1.95}, 2.9, 2.4, 0.81, {0, 1.16, 1.57}, 5.25, 4.4, 0.0038},
        {3, {0, 1.5, 2.35, 3.15}, 3.9, 1.3, 0.68, {0, 1.63, 2.20, 2.87}, 5.75, 4.7, 0.0048},
        {1, {0, 3.6}, 2.8, 1.3, 1.0, {0, 3.6}, 5.75, 5.7, 0.0099},
        // mixed
        {3, {0, 1.03, 1.3, 1.6}, 3.0, 2.6, 0.81, {0, 0.98, 1.13, 1.36}, 5.1, 4.2, 0.0027},
        {3, {0, 1.03, 1.3, 1.6}, 3.1, 2.2, 0.75, {0, 1.13, 1.34, 1.62}, 5.4, 4.4, 0.0031},
        {3, {0, 1.03, 1.3, 1.6}, 3.7, 1.1, 0.67, {0, 2.28, 2.82, 3.48}, 5.4, 5.3, 0.0057},
        // fixed axes (the runtime-shaped kernel; no blocks): FP64, mixed
        {3, {0, 1.98, 2.48, 3.83}},
        {4, {0, 1.66, 1.92, 2.21, 2.9}},
    };
    const Price& p = prices[gc.fixed ? 6 + f32 : 3 * f32 + (pow_law ? 2 : sat)];
    const int64_t tiles = (int64_t)((gc.n0 + v.bx - 1) / v.bx) * ((gc.n1 + v.by - 1) / v.by);
    const int64_t slots = 256 * p.per_cu;
    // rounds of nb workgroups, the last one mixed of itself and its share
    const auto rounds = [&](int64_t nb, const double* c, double mix) {
        const int64_t full = nb / slots, rem = nb % slots;
        if (!rem) return (double)full;
        const double share = (double)rem / slots, own = c[(rem + 255) / 256] / c[p.per_cu];
        return full ? full + mix * own + (1.0 - mix) * share : own;
    };
    int best = v.bz;
    double best_cost = INFINITY;
    for (int z = std::min(v.bz, gc.n2); z >= 1; --z) {
        const int nzc = (gc.n2 + z - 1) / z;
        const int bz = (gc.n2 + nzc - 1) / nzc;   // chunks of equal length
        if (bz != z) continue;
        const int64_t nb = tiles * nzc;
        const double late = pow_law || sat ? 0.0 : 0.15 * std::min(1.0, std::max(0.0, (double)nb / slots - 1.0));
        const double cost = (bz + 2) * (rounds(nb, p.chunk, 0.5) + late);
        if (cost < best_cost) {
            best_cost = cost;
            best = bz;
        }
    }
    v.bz = best;
    const int64_t N = (int64_t)gc.n0 * gc.n1 * gc.n2;
    if (gc.ndim == 3 && !gc.fixed && N < (int64_t)1 << 29 &&   // 32-bit byte offsets
        (N <= (int64_t)1 << 22 || (pow_law && !f32))) {
        Variant w{kBlockX, kBlockY, kBlockZ, 1};
        w.block = true;
        const double march = p.start + (best + p.lead) * p.it[p.per_cu] *
                                           rounds(tiles * ((gc.n2 + best - 1) / best), p.it, p.mix);
        // near a tie blocks were the faster ones (112^3, 65 x 65 x 300, 256 x 256 x 3 mixed)
        if (std::max(p.least, p.b0 + p.b1 * stage_blocks(w, gc)) < 1.03 * march) return w;
    }
    return v;
}

int64_t stage_blocks(Variant v, const GridConst& gc) {
    return (int64_t)((gc.n0 + v.bx - 1) / v.bx) * ((gc.n1 + v.by - 1) / v.by) * ((gc.n2 + v.bz - 1) / v.bz);
}

hipError_t launch_stage(int precision, Variant v, const GridConst& gc, int kind, int stage,
                        const double* Yin, const double* Ym2, const double* Y0, const void* MY0in,
                        void* MY0out, double* Yout, const void* b, const GridState* state,
                        const double* coef, hipStream_t st, double sub_scale, const Route* route,
                        const ExtOut* ext) {
    StageLaunch P;
    TileArgs& a = P.t;
    a.Yin = Yin;
    a.Ym2 = Ym2;
    a.Y0 = Y0;
    a.MY0in = MY0in;
    a.MY0out = MY0out;
    a.Yout = Yout;
    a.b = b;
    a.n0 = gc.n0;
    a.n1 = gc.n1;
    a.n2 = gc.n2;
    a.ndim = gc.ndim;
    a.x0 = a.y0 = a.z0 = a.z1 = 0;
    a.bx = v.bx;
    a.by = v.by;
    a.kind = kind;
    a.bc = gc.bc;
    a.fixed = gc.fixed;
    for (int i = 0; i < 6; ++i) a.gh[i] = gc.gh[i];
    a.ih0 = gc.ih0;
    a.ih1 = gc.ih1;
    a.ih2 = gc.ih2;
    a.scale = 0.0;
    a.mu = a.nu = a.omn = a.mut = a.gt = 0.0;
    a.ext = 0;
    // A grid whose stage fields (48 B a cell) about fit the 256 MB last-level
    // cache finds its pointwise fields there again in the next stage; larger ones
    // stream them past it, since they only displace the halo lines that tiles
    // share.  Mixed, us a stage, streamed / kept: 128^3 26.2 / 25.3, 150 x 127 x
    // 101 29.6 / 27.4, 160^3 43.8 / 40.6, 192^3 (340 MB) 64.3 / 62.1; 200^3 (384 MB)
    // 84.0 / 84.6, 208^3 81 / 88, 256^3 164 / 171.  In FP64 (64 B) 128^3 34.8 / 33.7
    // and 160^3 58.9 / 57.1, but 176^3 (349 MB) no longer: not built.
    P.cached = precision == RKL_MIXED && 48 * (int64_t)gc.n0 * gc.n1 * gc.n2 <= (int64_t)352 << 20;
    P.ntx = (gc.n0 + v.bx - 1) / v.bx;
    P.nty = (gc.n1 + v.by - 1) / v.by;
    P.bz = v.bz;
    const int nzc = (gc.n2 + v.bz - 1) / v.bz;
    P.state = state;
    P.coef = coef;
    P.stage = stage;
    P.kappa0 = gc.kappa0;
    P.kexp = gc.kexp;
    P.kperp = gc.kperp;
    P.satq = gc.satq;
    P.kmode = gc.kmode;
    P.fac = gc.fac;
    P.sub_scale = sub_scale;
    P.route = Route{nullptr, nullptr, 0, 0, 0};
    P.ext = ExtOut{nullptr, nullptr};
    if (ext) {
        // the last-stage extrema: routed RKL2 stages of 3-D grids without fixed axes
        if (!route || kind != 2 || gc.ndim != 3 || gc.fixed || !ext->part || !ext->ok) return hipErrorInvalidValue;
        P.ext = *ext;
    }
    if (route) {
        // routed stages: Yout carries the caller's T to the kernel
        if ((kind != 1 && kind != 2) || !route->A || !route->B || !Yout) return hipErrorInvalidValue;
        P.route = *route;
        a.Yin = Yout;
        a.Ym2 = Yout;
        a.Y0 = Yout;
    }
    const int64_t nb = (int64_t)P.ntx * P.nty * nzc;
    if (nb <= 0 || nb > 0x7fffffff) return hipErrorInvalidValue;
    const bool lim = gc.limiter != 0;
    const int sat = gc.saturation;
    if (precision == RKL_MIXED) return launch_prec<float>(P, (int)nb, v, lim, sat, st);
    return launch_prec<double>(P, (int)nb, v, lim, sat, st);
}

}  // namespace rkl
