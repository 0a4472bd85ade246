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

// ND: dimensions (1 or 2).  One cell per thread, three barriers a stage (two
// in 1-D).
template <typename R, bool LIM, int SAT, int KM, int ND>
__global__ __launch_bounds__(kFlatThreads) void flat_kernel(FlatLaunch P) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double rows[64 * 5];
    __shared__ double red[3][16];
    static_assert(kFlatThreads <= 16 * 64, "a slot of red per wave");
    __shared__ GridState sst;
    const int tid = threadIdx.x, nt = blockDim.x;
    const FlatTiling& t = P.t;
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
    const int tx = tid % w, ty = tid / w;
    const bool act = tx < w0 && ty < h1;
    const int slot = act ? tid : 0;
    const int gx = act ? lo0 + tx : lo0, gy = act ? lo1 + ty : lo1;
    const int cx = wrap(gx, n0), cy = wrap(gy, n1);
    const size_t c = (size_t)cy * n0 + cx;
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
    FaceDir<R> dx{0, 0, 0, 0, false}, dy{0, 0, 0, 0, false}, dl{0, 0, 0, 0, false};
    // the extra low face of this thread (edge of a non-periodic axis): faces
    // of the x edge first, then of the y edge
    const int jx = el0 ? h1 : 0, jy = ND == 2 && el1 ? w0 : 0;
    const bool job = tid < jx + jy, jobx = tid < jx;
    int jr = 0, jl = 0, jf = 0;   // slots of its two cells, place of its face
    if (act) {
        if (head) {
            y1 = P.T[c];
            y0 = y1;
        } else {
            y1 = P.in1[c];
            if (P.kind == 1) {
                y2 = P.in2[c];
                y0 = P.Y0c[c];
                my = ((const R*)P.M)[c];
            }
        }
        // beyond an outflow or fixed edge b repeats the edge cell's
        const size_t cxp = (size_t)cy * n0 + bidx(gx + 1, n0, ox), cyp = (size_t)bidx(gy + 1, n1, oy) * n0 + cx;
        const R u0 = b0[c], u1 = b1[c], u2 = b2[c];
        dx = face_dir(u0, u1, u2, b0[cxp], b1[cxp], b2[cxp]);
        if (ND == 2) dy = face_dir(u1, u0, u2, b1[cyp], b0[cyp], b2[cyp]);
    }
    if (job) {
        const int q = jobx ? tid : tid - jx;
        jr = jobx ? q * w : q;
        jl = jobx ? (fx ? gxl + q : jr) : (fy ? gyl + q : jr);
        jf = cells + q;
        const size_t e = jobx ? (size_t)wrap(lo1 + q, n1) * n0 : (size_t)wrap(lo0 + q, n0);
        const R u0 = b0[e], u1 = b1[e], u2 = b2[e];
        dl = jobx ? face_dir(u0, u1, u2, u0, u1, u2) : face_dir(u1, u0, u2, u1, u0, u2);
    }

    // dt_par, s and T_ref: the extrema of T, by every workgroup for itself
    if (P.derive) {
        block_state(P.gc, P.src, blockIdx.x == 0, P.state, red, &sst);
    } else {
        if (tid == 0) sst = *P.state;
        __syncthreads();
    }
    const int s = __builtin_amdgcn_readfirstlane(sst.s);
    const double tref = sizeof(R) == 4 ? uniform(sst.tref) : 0.0;
    const FaceK<R> fk = make_facek<R>(P.gc.kappa0, P.gc.kexp, P.gc.kperp, P.gc.satq, tref);
    int j0 = 1, j1 = 1;
    bool last = true;
    double scale = -P.gc.fac;
    if (P.kind == 1) {
        if (s < P.smin || s > P.s_cap) return;   // uniform over the launch
        const int G = P.groups ? P.groups : (t.nt0 * t.nt1 == 1 ? 1 : max(2, (s + t.f - 1) / t.f));
        j0 = (int)(((long long)s * P.group + G - 1) / G) + 1;
        j1 = (int)(((long long)s * (P.group + 1) + G - 1) / G);
        last = P.group == G - 1;
        scale = -uniform(sst.cdiv);
    } else if (P.kind == 2) {
        j1 = P.count;
        last = P.last != 0;
    }

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
        if (P.kind == 1 && (j - j0) % 64 == 0) {
            __syncthreads();   // the previous rows have been read
            const int nr = min(64, j1 - j + 1);
            if (P.coef) {
                for (int i = tid; i < 5 * nr; i += nt) rows[i] = P.coef[5 * ((size_t)s * (s + 1) / 2 + j) + i];
            } else if (tid < nr) {
                rkl2_row(s, j + tid, rows + 5 * tid);
            }
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

template <typename R, bool LIM, int SAT, int KM>
static void flat_nd(const FlatLaunch& P, size_t lds, hipStream_t st) {
    if (P.gc.ndim == 2) flat_kernel<R, LIM, SAT, KM, 2><<<P.t.blocks(), P.t.threads, lds, st>>>(P);
    else flat_kernel<R, LIM, SAT, KM, 1><<<P.t.blocks(), P.t.threads, lds, st>>>(P);
}
template <typename R, int SAT, int KM>
static void flat_lim(const FlatLaunch& P, size_t lds, hipStream_t st) {
    if (P.gc.limiter) flat_nd<R, true, SAT, KM>(P, lds, st);
    else flat_nd<R, false, SAT, KM>(P, lds, st);
}
template <typename R, int KM>
static void flat_sat(const FlatLaunch& P, size_t lds, hipStream_t st) {
    if (P.gc.saturation == 2) flat_lim<R, 2, KM>(P, lds, st);
    else if (P.gc.saturation == 1) flat_lim<R, 1, KM>(P, lds, st);
    else flat_lim<R, 0, KM>(P, lds, st);
}

template <typename R>
hipError_t launch_flat_r(const FlatLaunch& P, hipStream_t st) {
    const FlatTiling& t = P.t;
    // one cell, and one extra low face, per thread
    if (t.threads > kFlatThreads || t.w * t.h > t.threads || t.w + t.h > t.threads || t.f < 1 || P.gc.n2 != 1 ||
        P.gc.ndim > 2 || (P.kind == 2 && (P.count < 0 || P.count > kFlatEuler)))
        return hipErrorInvalidValue;
    const size_t lds = flat_lds<R>(t, P.gc.ndim, P.gc.fixed != 0);
    if (P.gc.kmode == 0) flat_sat<R, 0>(P, lds, st);
    else if (P.gc.kmode == 1) flat_sat<R, 1>(P, lds, st);
    else flat_sat<R, 2>(P, lds, st);
    return hipGetLastError();
}

}  // namespace rkl
