// rkl_flat_kernel.h -- the kernel of rkl_flat.h; included by the units that
// instantiate it, one per flux precision.
#pragma once
#include "../../include/rkl.h"
#include "rkl_flat.h"
#include "rkl_tile.h"

namespace rkl {

// LDS of a workgroup: T and, in 2-D, the two slopes of every region cell (and
// of the ghost cells beyond fixed edges), then the +x and +y faces of every
// region cell with the faces of the low edges behind them.
template <typename R>
inline size_t flat_lds(const FlatTiling& t, int ndim, bool fixed) {
    const size_t cells = (size_t)t.w * t.h, slots = cells + (fixed ? 2 * (size_t)(t.w + t.h) : 0);
    return sizeof(R) * (ndim == 2 ? 3 * slots + 2 * cells + t.w + t.h : slots + cells + t.h);
}

// the slope along an axis of one cell, all of whose neighbours are the cell
// itself: 0, or without the limiter NaN where t is not finite
template <typename R, bool LIM>
__device__ __forceinline__ R flat_slope(R t) {
    return LIM ? R(0) : t - t;
}

// the index of cell i of a periodic axis, -n <= i < 2n
__device__ __forceinline__ int wrap_once(int i, int n) {
    i = i < 0 ? i + n : i;
    return i >= n ? i - n : i;
}
// element i of a field of at most 2^26 cells: a scalar base and a 32-bit byte offset
template <typename E>
__device__ __forceinline__ E ld(const E* base, unsigned i) {
    return *(const E*)((const char*)base + i * (unsigned)sizeof(E));
}

// ND: dimensions (1 or 2).  One cell per thread, three barriers a stage (two
// in 1-D).  The state and every input are asked for before anything waits;
// ASK: s is asked for before everything else (flat_asks).
template <typename R, bool LIM, int SAT, int KM, int ND, bool ASK>
__global__ __launch_bounds__(kFlatThreads) void flat_kernel(FlatLaunch P) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double rows[64 * 5];
    __shared__ double red[3][16];
    static_assert(kFlatThreads <= 16 * 64, "a slot of red per wave");
    __shared__ GridState sst;
    const FlatTiling& t = P.t;
    if (ASK && P.group >= P.state->groups) return;
    const int tid = threadIdx.x, nt = blockDim.x;
    // the state as a former launch left it (the group that forms it does not use these)
    int s = P.state->s, G = P.state->groups;
    double tref = P.state->tref, cdiv = P.state->cdiv;
    const int n0 = P.gc.n0, n1 = P.gc.n1;
    const bool ox = P.gc.bc & 1, oy = P.gc.bc & 2, fx = P.gc.fixed & 1, fy = P.gc.fixed & 2;

    // the region and this thread's cell
    const int w = t.w, cells = t.w * t.h;
    const int tile0 = (int)blockIdx.x % t.nt0, tile1 = (int)blockIdx.x / t.nt0;
    const int halo = P.kind == 0 ? 1 : t.f;
    const int a0 = tile0 * t.o0, e0 = min(a0 + t.o0, n0);   // output tile
    const int a1 = tile1 * t.o1, e1 = min(a1 + t.o1, n1);
    const bool whole0 = t.nt0 == 1 && !ox, whole1 = t.nt1 == 1 && !oy;
    int lo0 = a0 - halo, hi0 = e0 + halo, lo1 = a1 - halo, hi1 = e1 + halo;
    if (t.nt0 == 1) { lo0 = 0; hi0 = n0; }
    else if (ox) { lo0 = max(lo0, 0); hi0 = min(hi0, n0); }
    if (t.nt1 == 1) { lo1 = 0; hi1 = n1; }
    else if (oy) { lo1 = max(lo1, 0); hi1 = min(hi1, n1); }
    const int w0 = hi0 - lo0, h1 = hi1 - lo1;
    // tid / w: the quotient is at least 0.5 / w from an integer, far more than its error
    const int ty = (int)(((float)tid + 0.5f) * __builtin_amdgcn_rcpf((float)w)), tx = tid - ty * w;
    const bool act = tx < w0 && ty < h1;
    const int slot = act ? tid : 0;
    const int gx = act ? lo0 + tx : lo0, gy = act ? lo1 + ty : lo1;
    const int cx = wrap_once(gx, n0), cy = wrap_once(gy, n1);   // a cut axis is longer than its halo
    const unsigned c = (unsigned)cy * n0 + cx;
    const bool store = act && gx >= a0 && gx < e0 && gy >= a1 && gy < e1;
    // the region ends at an edge of a non-periodic axis
    const bool el0 = ox && lo0 == 0, eh0 = ox && hi0 == n0, el1 = oy && lo1 == 0, eh1 = oy && hi1 == n1;
    // ghost slots behind the cells: x low, x high (h each), y low, y high (w each)
    const int gxl = cells, gxh = gxl + t.h, gyl = gxh + t.h, gyh = gyl + t.w;
    // slots of the neighbours.  At a cut border a cell stands in for the one
    // beyond it: its value there is wrong from the first stage on and reaches
    // one cell further in with each stage, F cells at most.
    int xm = slot - 1, xp = slot + 1, ym = slot - w, yp = slot + w;
    if (!act) xm = xp = ym = yp = slot;
    else {
        if (tx == 0) xm = whole0 ? slot + w0 - 1 : (el0 && fx ? gxl + ty : slot);
        if (tx == w0 - 1) xp = whole0 ? slot - (w0 - 1) : (eh0 && fx ? gxh + ty : slot);
        if (ty == 0) ym = whole1 ? slot + (h1 - 1) * w : (el1 && fy ? gyl + tx : slot);
        if (ty == h1 - 1) yp = whole1 ? slot - (h1 - 1) * w : (eh1 && fy ? gyh + tx : slot);
    }
    // where this cell's low faces are: the low neighbour's own +x / +y face,
    // or at a known edge an extra face
    const int fxl = act && tx == 0 && el0 ? cells + ty : (xm < cells ? xm : slot);
    const int fyl = act && ty == 0 && el1 ? cells + tx : (ym < cells ? ym : slot);

    const int slots = cells + (P.gc.fixed ? 2 * (t.w + t.h) : 0);
    R* LT = (R*)smem;
    R* SX = LT + slots;                              // 2-D only
    R* SY = SX + (ND == 2 ? slots : 0);
    R* FX = SY + (ND == 2 ? slots : 0);
    R* FY = FX + cells + t.h;                        // 2-D only

    // the cell's inputs and the directions of its +x and +y faces
    const size_t N = (size_t)n0 * n1;
    const R* b0 = (const R*)P.b;
    const R* b1 = b0 + N;
    const R* b2 = b1 + N;
    const bool head = P.kind != 1 ? P.first != 0 : P.group == 0;
    double y1 = 0.0, y2 = 0.0, y0 = 0.0;
    R my = 0;
    // the extra low face of this thread (edge of a non-periodic axis): faces
    // of the x edge first, then of the y edge
    const int jx = el0 ? h1 : 0, jy = ND == 2 && el1 ? w0 : 0;
    const bool job = tid < jx + jy, jobx = tid < jx;
    int jr = 0, jl = 0, jf = 0;   // slots of its two cells, place of its face
    if (head) {
        y1 = ld(P.T, c);
        y0 = y1;
    } else {
        y1 = ld(P.in1, c);
        if (P.kind == 1) {
            y2 = ld(P.in2, c);
            y0 = ld((const double*)P.Y0c, c);
            my = ld((const R*)P.M, c);
        }
    }
    // beyond an outflow or fixed edge b repeats the edge cell's
    const unsigned cxp = (unsigned)cy * n0 + (ox ? min(gx + 1, n0 - 1) : wrap_once(gx + 1, n0));
    const unsigned cyp = (unsigned)(oy ? min(gy + 1, n1 - 1) : wrap_once(gy + 1, n1)) * n0 + cx;
    const R u0 = ld(b0, c), u1 = ld(b1, c), u2 = ld(b2, c);
    const R x0 = ld(b0, cxp), x1 = ld(b1, cxp), x2 = ld(b2, cxp);
    R v0 = 0, v1 = 0, v2 = 0, e0b = 0, e1b = 0, e2b = 0;
    if (ND == 2) {
        v0 = ld(b0, cyp);
        v1 = ld(b1, cyp);
        v2 = ld(b2, cyp);
    }
    if (job) {
        const int q = jobx ? tid : tid - jx;
        jr = jobx ? q * w : q;
        jl = jobx ? (fx ? gxl + q : jr) : (fy ? gyl + q : jr);
        jf = cells + q;
        const unsigned e = jobx ? (unsigned)wrap_once(lo1 + q, n1) * n0 : (unsigned)wrap_once(lo0 + q, n0);
        e0b = ld(b0, e);
        e1b = ld(b1, e);
        e2b = ld(b2, e);
    }

    // dt_par, s and T_ref: the extrema of T, by every workgroup for itself
    if (P.derive) {
        block_state(P.gc, P.src, blockIdx.x == 0, P.state, red, &sst);
        s = __builtin_amdgcn_readfirstlane(sst.s);
        tref = uniform(sst.tref);
        cdiv = uniform(sst.cdiv);
    }
    if (sizeof(R) == 8) tref = 0.0;
    int j0 = 1, j1 = 1;
    bool last = true;
    double scale = -P.gc.fac;
    if (P.kind == 1) {
        if (P.derive) {
            if (s < P.smin || s > P.s_cap) return;   // uniform over the launch; groups stays 0
            G = s >= P.s_even ? P.launches : flat_groups(t, s);
            if (blockIdx.x == 0 && tid == 0) P.state->groups = G;
        } else if (P.group >= G) {
            return;
        }
        j0 = (int)(((unsigned)s * P.group + G - 1) / G) + 1;
        j1 = (int)(((unsigned)s * (P.group + 1) + G - 1) / G);
        last = P.group == G - 1;
        scale = -cdiv;
    } else if (P.kind == 2) {
        j1 = P.count;
        last = P.last != 0;
    }
    // the coefficient rows of up to 64 stages
    const auto fill_rows = [&](int j) {
        const int nr = min(64, j1 - j + 1);
        if (P.coef) {
            for (int i = tid; i < 5 * nr; i += nt) rows[i] = P.coef[5 * ((size_t)s * (s + 1) / 2 + j) + i];
        } else if (tid < nr) {
            rkl2_row(s, j + tid, rows + 5 * tid);
        }
    };
    if (P.kind == 1) fill_rows(j0);
    const FaceK<R> fk = make_facek<R>(P.gc.kappa0, P.gc.kexp, P.gc.kperp, P.gc.satq, tref);
    const FaceDir<R> dx = face_dir(u0, u1, u2, x0, x1, x2);
    FaceDir<R> dy{0, 0, 0, 0, false}, dl{0, 0, 0, 0, false};
    if (ND == 2) dy = face_dir(u1, u0, u2, v1, v0, v2);
    if (job) dl = jobx ? face_dir(e0b, e1b, e2b, e0b, e1b, e2b) : face_dir(e1b, e0b, e2b, e1b, e0b, e2b);

    const R ih0 = R(P.gc.ih0), ih1 = R(P.gc.ih1);
    const R hih0 = R(0.25 * P.gc.ih0), hih1 = R(0.25 * P.gc.ih1);   // 1/(4h), see cell_slope
    if (act) LT[slot] = to_r<R>(y1, tref);
    // the ghost cells beyond fixed edges: temperatures and transverse slopes
    // that hold for every stage
    if (P.gc.fixed) {
        const auto gt = [&](int i, int j) -> R {
            const GhostCol g = ghost_col(P.gc.bc, P.gc.fixed, P.gc.gh, n0, n1, i, j);
            return to_r<R>(ghost_T(g, P.T, 0, 1, false, false, 0, N), tref);
        };
        for (int q = tid; q < 2 * (t.w + t.h); q += nt) {
            const bool gxq = q < 2 * t.h;
            const int k = gxq ? q % t.h : (q - 2 * t.h) % t.w;
            const bool high = gxq ? q >= t.h : q >= 2 * t.h + t.w;
            if (gxq ? !(fx && k < h1 && (high ? eh0 : el0)) : !(fy && k < w0 && (high ? eh1 : el1))) continue;
            const int i = gxq ? (high ? n0 : -1) : lo0 + k, j = gxq ? lo1 + k : (high ? n1 : -1);
            const R g = gt(i, j);
            LT[cells + q] = g;
            if (ND == 2) {
                if (gxq) SY[cells + q] = cell_slope<R, LIM>(gt(i, j - 1), g, gt(i, j + 1), hih1);
                else SX[cells + q] = cell_slope<R, LIM>(gt(i - 1, j), g, gt(i + 1, j), hih0);
            }
        }
    }

    double tl = 0.0;
    for (int j = j0; j <= j1; ++j) {
        if (P.kind == 1 && j > j0 && (j - j0) % 64 == 0) {
            __syncthreads();   // the previous rows have been read
            fill_rows(j);
        }
        __syncthreads();
        const R tc = LT[slot];
        R sx = 0, sy = 0;
        if (ND == 2) {
            sx = cell_slope<R, LIM>(LT[xm], tc, LT[xp], hih0);
            sy = cell_slope<R, LIM>(LT[ym], tc, LT[yp], hih1);
            if (act) {
                SX[slot] = sx;
                SY[slot] = sy;
            }
            __syncthreads();
        }
        const R zc = flat_slope<R, LIM>(tc);
        R f0, f1 = 0;
        {
            const R tr = LT[xp], zr = flat_slope<R, LIM>(tr);
            const R z = face_transverse<R, LIM>(zc, zr);
            f0 = face_flux_dir<R, SAT, KM>(tc, tr, ih0, ND == 2 ? face_transverse<R, LIM>(sy, SY[xp]) : z, z, dx, fk);
            if (act) FX[slot] = f0;
        }
        if (ND == 2) {
            const R tr = LT[yp], zr = flat_slope<R, LIM>(tr);
            f1 = face_flux_dir<R, SAT, KM>(tc, tr, ih1, face_transverse<R, LIM>(sx, SX[yp]),
                                           face_transverse<R, LIM>(zc, zr), dy, fk);
            if (act) FY[slot] = f1;
        }
        if (job) {
            const R ta = LT[jl], tb = LT[jr];
            const R z = face_transverse<R, LIM>(flat_slope<R, LIM>(ta), flat_slope<R, LIM>(tb));
            R g1 = z;
            if (ND == 2) {
                const R* S = jobx ? SY : SX;
                g1 = face_transverse<R, LIM>(S[jl], S[jr]);
            }
            const R f = face_flux_dir<R, SAT, KM>(ta, tb, jobx ? ih0 : ih1, g1, z, dl, fk);
            if (jobx) FX[jf] = f;
            else FY[jf] = f;
        }
        __syncthreads();
        R div = (f0 - FX[fxl]) * ih0;
        if (ND == 2) div = fma(f1 - FY[fyl], ih1, div);
        if (P.kind == 1) {
            tl = scale * (double)div;
            const double* cf = rows + 5 * ((j - j0) % 64);
            double y;
            if (j == 1) {
                my = R(tl);
                y = fma(cf[3], (double)my, y1);
            } else {
                y = stage_combine(cf[0], cf[1], cf[2], cf[3], cf[4], y1, y2, y0, tl, (double)my);
            }
            y2 = y1;
            y1 = y;
        } else if (P.kind == 2) {
            y1 = y1 + P.scale[j - 1] * (double)div;
        } else {
            tl = scale * (double)div;
        }
        if (act) LT[slot] = to_r<R>(y1, tref);
    }

    if (!store) return;
    if (P.kind == 0) {
        P.Tout[c] = tl;
    } else if (last) {
        P.Tout[c] = y1;
    } else {
        P.out1[c] = y1;
        if (P.kind == 1) {
            P.out2[c] = y2;
            if (P.group == 0) {
                P.Y0c[c] = y0;
                ((R*)P.M)[c] = my;
            }
        }
    }
}

template <typename R, bool LIM, int SAT, int KM, int ND>
static void flat_ask(const FlatLaunch& P, size_t lds, hipStream_t st, bool ask) {
    if (ask) flat_kernel<R, LIM, SAT, KM, ND, true><<<P.t.blocks(), P.t.threads, lds, st>>>(P);
    else flat_kernel<R, LIM, SAT, KM, ND, false><<<P.t.blocks(), P.t.threads, lds, st>>>(P);
}
template <typename R, bool LIM, int SAT, int KM>
static void flat_nd(const FlatLaunch& P, size_t lds, hipStream_t st, bool ask) {
    if (P.gc.ndim == 2) flat_ask<R, LIM, SAT, KM, 2>(P, lds, st, ask);
    else flat_ask<R, LIM, SAT, KM, 1>(P, lds, st, ask);
}
template <typename R, int SAT, int KM>
static void flat_lim(const FlatLaunch& P, size_t lds, hipStream_t st, bool ask) {
    if (P.gc.limiter) flat_nd<R, true, SAT, KM>(P, lds, st, ask);
    else flat_nd<R, false, SAT, KM>(P, lds, st, ask);
}
template <typename R, int KM>
static void flat_sat(const FlatLaunch& P, size_t lds, hipStream_t st, bool ask) {
    if (P.gc.saturation == 2) flat_lim<R, 2, KM>(P, lds, st, ask);
    else if (P.gc.saturation == 1) flat_lim<R, 1, KM>(P, lds, st, ask);
    else flat_lim<R, 0, KM>(P, lds, st, ask);
}

template <typename R>
hipError_t launch_flat_r(const FlatLaunch& P, hipStream_t st, bool ask) {
    const FlatTiling& t = P.t;
    // one cell, and one extra low face, per thread
    if (t.threads > kFlatThreads || t.w * t.h > t.threads || t.w + t.h > t.threads || t.f < 1 || P.gc.n2 != 1 ||
        P.gc.ndim > 2 || (P.kind == 2 && (P.count < 0 || P.count > kFlatEuler)))
        return hipErrorInvalidValue;
    const size_t lds = flat_lds<R>(t, P.gc.ndim, P.gc.fixed != 0);
    if (P.gc.kmode == 0) flat_sat<R, 0>(P, lds, st, ask);
    else if (P.gc.kmode == 1) flat_sat<R, 1>(P, lds, st, ask);
    else flat_sat<R, 2>(P, lds, st, ask);
    return hipGetLastError();
}

}  // namespace rkl
