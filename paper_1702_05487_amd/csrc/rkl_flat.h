// rkl_flat.h -- several stages per launch on 1-D and 2-D grids (gfx950).
// Private to librkl.
//
// Method: Vaidya et al. (2017), arXiv:1702.05487, Appendix A (RKL2, and RKL1
// of Sec. 3.3) and the explicit sub-steps of Sec. 2.3, with the face flux of
// rkl_tile.h.
//
// What bounds it: a 1-D or 2-D stage of these grids is a few hundred
// nanoseconds of arithmetic, so one launch per stage spends its time on the
// launch itself (2.6 us for an empty one) and on filling the pipeline.  Here
// a workgroup holds a region of the grid, one cell per thread, for F stages:
// the stage values of the cell stay in registers, the input and its slopes in
// LDS, and the field directions of its faces are formed once.  A region
// reaches F cells beyond its output tile (each stage needs one cell around
// it, including the corners), except at edges the region itself knows: an
// outflow or fixed edge, or a periodic axis that lies in the region whole.
// The cells of the border are computed by the neighbouring workgroups too.
//
// A super-step of s stages is cut into G groups of at most F stages, one
// launch each.  Group 0 reads T, takes dt_par, s and T_ref (from T itself or
// from the reduction's partial extrema, each workgroup for itself) and keeps
// tau M(Y0) and a copy of Y0; each group hands Y_j and Y_{j-1} on in a pair of
// buffers that it does not read; the last writes T, which no workgroup of its
// launch reads.  So G >= 2, unless one workgroup holds the whole grid.
// Every operation is that of run_tile, so the results have its bits.
#pragma once
#include "rkl_internal.h"

namespace rkl {

constexpr int kFlatThreads = 1024;   // most threads (and cells) of a workgroup
constexpr int kFlatEuler = 64;       // most sub-steps of one Euler launch
constexpr int64_t kFlatMostCells = int64_t(1) << 26;   // larger grids run one stage a launch

// How a 1-D or 2-D grid is cut: regions of at most w x h cells, output tiles
// of o0 x o1 cells, at most f stages a launch.
struct FlatTiling {
    int w = 0, h = 0, o0 = 0, o1 = 0, nt0 = 0, nt1 = 0, f = 0;
    int threads = 0;
    int blocks() const { return nt0 * nt1; }
};
// the tiling for grid gc (1-D or 2-D), or f = 0 where one launch per stage is used;
// few: for super-steps of at most kFewStages
FlatTiling flat_tiling(int precision, const GridConst& gc, bool few = false);
// Stage counts with a tiling of their own on 2-D grids of 2^16 cells and more: the
// ordinary one reaches f cells around each tile, which pays from about five stages
// on.  s = 3, us a super-step, one stage a launch / ordinary / few: 2048^2 mixed
// (kappa0) 305 / 338 / 250, mixed T^1.7 396 / 458 / 406, FP64 T^2.5 450 / 355 / 303.
constexpr int kFewStages = 4;
inline bool flat_is_few(const GridConst& gc, int64_t stages) {
    return gc.ndim == 2 && stages <= kFewStages && (int64_t)gc.n0 * gc.n1 >= 65536;
}
// the tiling of a single operator evaluation
FlatTiling flat_tiling_once(int precision, const GridConst& gc);
// groups of a super-step of s stages
__host__ __device__ inline int flat_groups(const FlatTiling& t, int s) {
    if (t.nt0 * t.nt1 == 1) return 1;
    const int g = (s + t.f - 1) / t.f;
    return g < 2 ? 2 : g;
}

// A super-step of s stages with `launches` enqueued before s is known spreads
// its stages evenly over all of them while they are at most twice what it needs
// (one without stages costs about as much as the set-up of one with few), that
// is from this s on; below it is cut into the groups it needs.
inline int flat_even_from(const FlatTiling& t, int launches, int smin) {
    const int half = (launches + 1) / 2;
    return half <= 2 ? smin : t.f * (half - 1) + 1;
}

// Super-steps with s on the device: whether launch `group` asks for s before it
// loads anything.  It then costs 2 to 4 us where s has no such group, against a
// pass over the fields (1024 x 1024: 20 us), and 0.7 us (a small grid) to 17 us
// (2048 x 2048) more where it has.  So only the groups past 64 stages do.
inline bool flat_asks(const FlatTiling& t, int group) { return group > 1 && group >= flat_groups(t, 64); }

struct FlatLaunch {
    int kind;            // 0 flux divergence, 1 super-step group, 2 Euler sub-steps
    const double* T;     // Y0: the stencil input of group 0
    double* Tout;        // kind 0: out; else T, written by the last group
    double* Y0c;         // copy of Y0, written by group 0
    void* M;             // tau M(Y0), type R
    const double* in1;   // groups >= 1: Y_{j0-1}
    const double* in2;   //              Y_{j0-2}
    double* out1;        // groups before the last: Y_{j1}
    double* out2;        //                         Y_{j1-1}
    const void* b;
    GridState* state;
    const double* coef;  // RKL table, row (s, j) at 5 (s(s+1)/2 + j); NULL: RKL2 rows formed here
    int group;           // nothing is done from state->groups on, which group 0 stores:
    int launches;        // `launches` from s_even stages on, else flat_groups(t, s);
    int s_even;
    int smin, s_cap;     // 0 where s is outside [smin, s_cap]
    FlatTiling t;
    GridConst gc;
    int derive;          // every workgroup forms the state from src; else *state holds it
    StateSource src;
    int first, last;     // kind 2: the first reads T, the last writes Tout
    int count;           // kind 2: sub-steps of this launch
    double scale[kFlatEuler];   // kind 2: -tau_k (gamma-1)/rho
};

hipError_t launch_flat(int precision, const FlatLaunch& P, hipStream_t st, bool ask = false);   // ask: see flat_asks
template <typename R>
hipError_t launch_flat_r(const FlatLaunch& P, hipStream_t st, bool ask);
extern template hipError_t launch_flat_r<float>(const FlatLaunch&, hipStream_t, bool);
extern template hipError_t launch_flat_r<double>(const FlatLaunch&, hipStream_t, bool);

}  // namespace rkl
