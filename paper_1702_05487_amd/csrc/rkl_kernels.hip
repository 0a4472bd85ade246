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
// before z0 fill the rings); an iteration takes c[k] microseconds with k
// workgroups on a CU (MC, T^2.5 and saturated flux; measured with 64^3 to
// 192^3 grids, k = 1, 2, 3; three mixed, two FP64 or three saturated FP64
// workgroups fit a CU's registers), and a launch 4 us besides.  Short chunks
// give a small grid enough workgroups for the 256 CUs, long ones keep the two
// extra iterations and the halo planes cheap.  The last, partly filled round is priced half by its share
// of the slots and half as a round of its own: workgroups of different rounds
// overlap, but not fully.
//
// Blocks of 16 x 4 x 4 cells (rkl_block.h): no march, so the least a launch
// takes is 5.4 us (FP64; mixed 5.0), but 0.0056 us (0.0035) more per block
// against 0.0025 (0.0016) for 256 marched cells of a large grid.
//
// Measured per stage, 32-plane chunks / the chunk taken here / blocks:
// 45 x 33 x 29 FP64 37.8 / 9.0 / 5.5 us, 64^3 mixed 38.0 / 9.4 / 7.4 us, 64^3
// FP64 49.3 / 12.5 / 9.8 us, 96^3 FP64 49.9 / 23.5 / 24.1 us, 128^3 FP64 50.7 /
// 42.4 / 50.1 us, 150 x 127 x 101 mixed 45.2 / 30.3 / 33.4 us.
Variant fit_variant(int precision, Variant v, const GridConst& gc) {
    if (gc.fixed) {
        v.bx = v.by = 16;   // the tile shape of the ghost-loading kernel
        v.fuse = 1;
    }
    if (v.exact) return v;
    const bool f32 = precision == RKL_MIXED;
    const bool three = !f32 && gc.saturation && gc.kmode != 2 && !gc.fixed && v.bx != 64;   // as three_waves
    const int per_cu = f32 || three ? 3 : 2;
    static const double c32[] = {0.0, 1.03, 1.3, 1.6}, c64[] = {0.0, 1.3, 1.95},
                        c64s[] = {0.0, 1.5, 2.35, 3.15};
    const double* c = f32 ? c32 : three ? c64s : c64;
    const int64_t tiles = (int64_t)((gc.n0 + v.bx - 1) / v.bx) * ((gc.n1 + v.by - 1) / v.by);
    const int64_t slots = 256 * per_cu;
    int best = v.bz;
    double best_cost = INFINITY;
    for (int z = std::min(v.bz, gc.n2); z >= 1; --z) {
        const int nzc = (gc.n2 + z - 1) / z;
        const int bz = (gc.n2 + nzc - 1) / nzc;   // chunks of equal length
        if (bz != z) continue;
        const int64_t nb = tiles * nzc, full = nb / slots, rem = nb % slots;
        double rounds = (double)full;
        if (rem) {
            const double share = (double)rem / slots, own = c[(rem + 255) / 256] / c[per_cu];
            rounds += full ? 0.5 * (share + own) : own;
        }
        const double cost = (bz + 2) * rounds;
        if (cost < best_cost) {
            best_cost = cost;
            best = bz;
        }
    }
    v.bz = best;
    if (gc.ndim == 3 && !gc.fixed && (int64_t)gc.n0 * gc.n1 * gc.n2 < (int64_t)1 << 29) {   // 32-bit byte offsets
        Variant w{kBlockX, kBlockY, kBlockZ, 1};
        w.block = true;
        const double nb = (double)stage_blocks(w, gc);
        const double block = f32 ? std::max(5.0, 4.0 + 0.0035 * nb) : std::max(5.4, 4.1 + 0.0056 * nb);
        if (block < 4.0 + c[per_cu] * best_cost) return w;
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
