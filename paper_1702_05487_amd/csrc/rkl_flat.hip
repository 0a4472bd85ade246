// rkl_flat.hip -- how 1-D and 2-D grids are cut into the regions of
// rkl_flat.h, and the launch by flux precision.
#include "rkl_flat.h"

#include <algorithm>
#include <cmath>

#include "../../include/rkl.h"

namespace rkl {

// Microseconds per stage of a grid cut by tiling t.  Measured (one MI355X, 20
// back-to-back super-steps): a launch costs about 2 us, each round of resident
// workgroups 2.2 us (1-D) or 4 us (2-D) of loads and set-up, and a stage 0.45 us
// of dependent latency plus the issue time of the waves that share a SIMD,
// which grows with the work of a face.  The registers allow four waves per
// SIMD, one workgroup of 1024 threads.  The stage count is not known here, and
// several regions take two launches at least, so no more than 10 (1-D: 14)
// stages are priced together; one region runs all stages (24 priced) at once.
// Measured per super-step against one stage per launch: 400 cells (s = 20)
// 120 -> 17 us, 64 x 64 (14) 85 -> 23 us, 200 x 200 MC (20) 130 -> 42 us;
// 1024 x 1024 mixed, MC and saturation, 34.7 -> 18.3 us per stage.
// (2 with `few`: two groups of at most two stages.)
static double flat_cost(int precision, const GridConst& gc, const FlatTiling& t, bool few) {
    const bool f32 = precision == RKL_MIXED, sat = gc.saturation != 0, lim = gc.limiter != 0;
    const bool km1 = gc.kmode == 1, km2 = gc.kmode == 2, two = gc.ndim == 2;
    const double face = !two ? (f32 ? 0.04 + 0.03 * sat : 0.05 + 0.05 * sat) + (km2 ? 0.2 : 0.0)
                        : f32 ? 2 * (0.05 + 0.03 * lim + 0.05 * sat + 0.03 * km1 + 0.1 * km2)
                              : 2 * (0.08 + 0.03 * lim + 0.08 * sat + 0.06 * km1 + 0.3 * km2);
    const double setup = two ? 4.0 : 2.2;
    const int f = t.blocks() == 1 ? 24 : std::min(t.f, few ? 2 : two ? 10 : 14);
    const int waves = t.threads / 64, per_cu = std::max(1, 16 / waves);
    const int64_t nb = t.blocks(), slots = 256 * per_cu, full = nb / slots, rem = nb % slots;
    const auto round = [&](int64_t wgs) { return setup + f * (0.45 + face * ((wgs * waves + 3) / 4)); };
    double tm = 2.0 + full * round(per_cu);
    if (rem) tm += round((rem + 255) / 256);
    return tm / f;
}

static int round64(int x) { return (x + 63) / 64 * 64; }

// regions of at most w x h cells with room for f stages; f = 0 where they do
// not fit the threads or the LDS of a workgroup
static FlatTiling shape(const GridConst& gc, int w, int h, int f) {
    FlatTiling t;
    if (gc.n0 <= w) { t.w = t.o0 = gc.n0; t.nt0 = 1; }
    else { t.w = w; t.o0 = w - 2 * f; }
    if (gc.n1 <= h) { t.h = t.o1 = gc.n1; t.nt1 = 1; }
    else { t.h = h; t.o1 = h - 2 * f; }
    if (t.o0 < 1 || t.o1 < 1) return FlatTiling();
    t.nt0 = (gc.n0 + t.o0 - 1) / t.o0;
    t.nt1 = (gc.n1 + t.o1 - 1) / t.o1;
    if ((int64_t)t.nt0 * t.nt1 > 0x7fffffff) return FlatTiling();
    t.threads = round64(std::max(t.w * t.h, t.w + t.h));
    if (t.threads > kFlatThreads) return FlatTiling();
    const size_t es = 8, cells = (size_t)t.w * t.h, slots = cells + (gc.fixed ? 2 * (size_t)(t.w + t.h) : 0);
    if (es * (gc.ndim == 2 ? 3 * slots + 2 * cells + t.w + t.h : slots + cells + t.h) > 60000) return FlatTiling();
    t.f = f;
    return t;
}

FlatTiling flat_tiling(int precision, const GridConst& gc, bool few) {
    FlatTiling best;
    if (gc.ndim > 2 || gc.n2 != 1) return best;
    double cost = INFINITY;
    const auto take = [&](int w, int h, int f) {
        const FlatTiling t = shape(gc, w, h, f);
        if (!t.f) return;
        const double c = flat_cost(precision, gc, t, few);
        if (c < cost) {
            cost = c;
            best = t;
        }
    };
    // one region: every stage in one launch
    if ((int64_t)gc.n0 * gc.n1 <= kFlatThreads) take(gc.n0, gc.n1, kFlatEuler);
    if (gc.ndim == 1) {
        for (int w : {256, 512, 1008})
            for (int f = 1; f <= kFlatEuler && 2 * f < w; ++f) take(w, 1, f);
    } else {
        static const int shapes[][2] = {{16, 16}, {24, 24}, {32, 16}, {32, 24}, {32, 32}, {64, 16}};
        for (const auto& q : shapes)
            for (int f = 1; 2 * f < std::max(q[0], q[1]); ++f) take(q[0], q[1], f);
    }
    return best;
}

FlatTiling flat_tiling_once(int precision, const GridConst& gc) {
    FlatTiling t;
    if (gc.ndim > 2 || gc.n2 != 1) return t;
    t = gc.ndim == 1 ? shape(gc, 256, 1, 1) : shape(gc, 32, 16, 1);
    return t;
}

hipError_t launch_flat(int precision, const FlatLaunch& P, hipStream_t st, bool ask) {
    return precision == RKL_MIXED ? launch_flat_r<float>(P, st, ask) : launch_flat_r<double>(P, st, ask);
}

}  // namespace rkl
