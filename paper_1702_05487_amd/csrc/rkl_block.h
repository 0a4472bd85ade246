// rkl_block.h -- the one-stage kernel of small 3-D grids (gfx950): a workgroup
// computes a block of 16 x 4 x 4 cells at once instead of marching along z.
// Private to librkl; included by the units that instantiate it.
//
// What bounds it: the latency of one stage.  The z-march of run_tile needs at
// least three dependent plane iterations, each 1.0-1.3 us with one workgroup
// on a CU, and is hidden only by other workgroups; a grid of some 10^4 cells
// has none.  Here every load is issued at once and the stage is three phases
// (slopes; faces; divergence and recurrence) between barriers, with all slopes
// and all faces of the block in parallel.  It loads and slopes more halo per
// cell (392 ring cells for 256), which large grids would pay for.
// The operations on each cell and face are run_tile's: same bits.
//
// A routed launch beyond s that only finds out when the state has arrived has
// by then asked for every field: 64^3 4 us, 96^3 FP64 12.6 us, 140 x 130 x 120
// 29 us, instead of 2.2, 3.1 and 5.6 us where it asks for s first (ASK).  With
// more than four blocks per CU others hide that wait, and stages past 64 are
// rarely all needed; otherwise it would cost a stage of 7 us 0.25 us.
#pragma once
#include "rkl_stage.h"

namespace rkl {

// One axis of n cells: the index of cell i, i in [-1, n] (beyond that any
// index in range: no stored cell depends on it).
struct NearAxis {
    int n, lo, hi;   // the cells standing in for -1 and n
    __device__ __forceinline__ NearAxis(int n_, bool open) : n(n_), lo(open ? 0 : n_ - 1), hi(open ? n_ - 1 : 0) {}
    __device__ __forceinline__ int operator()(int i) const {
        const int c = i < n ? i : hi;
        return i < 0 ? lo : c;
    }
};
// element i of a field of fewer than 2^29 cells: a scalar base and a 32-bit
// byte offset, so that an address costs one shift
template <typename E>
__device__ __forceinline__ E ld(const E* base, unsigned i) {
    return *(const E*)((const char*)base + (i * (unsigned)sizeof(E)));
}

template <typename R, bool LIM, int SAT, int KM, bool ASK>
__global__ __launch_bounds__(256) void block_kernel(StageLaunch P) {
    constexpr int BX = kBlockX, BY = kBlockY, BZ = kBlockZ;
    static_assert(BX == 16 && BY == 4 && BZ == 4, "one 64-lane wave per z plane, and per y row of all planes");
    constexpr int PX = BX + 2, PP = PX * (BY + 2), PL = PP * (BZ + 2);
    __shared__ R LT[PL], LS[3][PL];
    __shared__ R FX[BZ * BY * (BX + 1)], FY[BZ * (BY + 1) * BX], FZ[(BZ + 1) * BY * BX];
    int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = bid % P.ntx * BX;
    bid /= P.ntx;
    const int y0 = bid % P.nty * BY, z0 = bid / P.nty * BZ;
    TileArgs a = P.t;
    stage_inputs(P, a);
    if (ASK && P.stage > P.state->s) return;
    const int s = P.state->s;
    const double cdiv = P.state->cdiv, tref = sizeof(R) == 4 ? P.state->tref : 0.0;
    const int n0 = a.n0, n1 = a.n1;
    const NearAxis X(n0, a.bc & 1), Y(n1, a.bc & 2), Z(a.n2, a.bc & 4);
    const size_t N = (size_t)n0 * n1 * a.n2;
    const R* b0 = (const R*)a.b;
    const R* b1 = b0 + N;
    const R* b2 = b1 + N;
    const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const auto at = [&](int gx, int gy, int gz) { return (unsigned)((gz * n1 + gy) * n0 + gx); };
    const auto slot = [](int x, int y, int z) { return ((z + 1) * (BY + 2) + y + 1) * PX + x + 1; };

    // every load of the block, issued before the state is known: T with its
    // ring, b of the own cell and of the cells its faces touch, the pointwise
    // stage inputs
    double tv[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        // q / 18 and q / 108 by 24-bit products, exact for q < 768
        const unsigned q = tid + 256 * i, row = q * 3641u >> 16, pl = q * 607u >> 16;
        if (i < 2 || q < PL)
            tv[i] = ld(a.Yin, at(X(x0 - 1 + (int)(q - PX * row)), Y(y0 - 1 + (int)(row - (BY + 2) * pl)),
                                 Z(z0 - 1 + (int)pl)));
    }
    const int tx = tid % BX, ty = tid / BX % BY, tz = tid / (BX * BY);
    const int gx = X(x0 + tx), gy = Y(y0 + ty), gz = Z(z0 + tz);
    const unsigned o = at(gx, gy, gz);
    const bool store = x0 + tx < n0 && y0 + ty < n1 && z0 + tz < a.n2;
    const double yk = ld(a.Yin, o);
    double ym2 = 0.0, yz = 0.0;
    R my0 = 0;
    if (a.kind == 2) {
        ym2 = ld(a.Ym2, o);
        yz = ld(a.Y0, o);
        my0 = ld((const R*)a.MY0in, o);
    }
    FaceDir<R> dx, dy, dz;
    {
        const R u0 = ld(b0, o), u1 = ld(b1, o), u2 = ld(b2, o);
        const unsigned ex = at(X(x0 + tx + 1), gy, gz), ey = at(gx, Y(y0 + ty + 1), gz), ez = at(gx, gy, Z(z0 + tz + 1));
        dx = face_dir(u0, u1, u2, ld(b0, ex), ld(b1, ex), ld(b2, ex));
        dy = face_dir(u1, u0, u2, ld(b1, ey), ld(b0, ey), ld(b2, ey));
        dz = face_dir(u2, u0, u1, ld(b2, ez), ld(b0, ez), ld(b1, ez));
    }
    // low faces of the block, one kind per wave: z (wave 0), y (wave 2), x (16
    // lanes of wave 3); jx, jy, jz: the cell above the face
    const bool jobz = wave == 0, joby = wave == 2, jobx = wave == 3;
    const bool job = jobz || joby || (jobx && lane < BY * BZ);
    const int jx = jobx ? 0 : lane % BX, jy = jobz ? lane / BX : jobx ? lane % BY : 0,
              jz = joby ? lane / BX : jobx ? lane / BY % BZ : 0;
    R r0 = 0, r1 = 0, r2 = 0, l0 = 0, l1 = 0, l2 = 0;
    if (job) {
        const int hx = X(x0 + jx), hy = Y(y0 + jy), hz = Z(z0 + jz);
        const unsigned r = at(hx, hy, hz),
                       l = at(jobx ? X(x0 - 1) : hx, joby ? Y(y0 - 1) : hy, jobz ? Z(z0 - 1) : hz);
        r0 = ld(b0, r); r1 = ld(b1, r); r2 = ld(b2, r);
        l0 = ld(b0, l); l1 = ld(b1, l); l2 = ld(b2, l);
    }
    if (!stage_args<true>(P, true, s, cdiv, a)) return;
    const FaceK<R> fk = make_facek<R>(P.kappa0, P.kexp, P.kperp, P.satq, tref);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int q = tid + 256 * i;
        if (i < 2 || q < PL) LT[q] = to_r<R>(tv[i], tref);
    }
    __syncthreads();

    // slopes of the own cells, and the two transverse ones of the ring cells
    // that share a face with the block: z low, z high, y low, y high (one
    // plane of 64 per wave), x low and high on wave 1
    const R ih0 = R(a.ih0), ih1 = R(a.ih1), ih2 = R(a.ih2);
    const R hih0 = R(0.25 * a.ih0), hih1 = R(0.25 * a.ih1), hih2 = R(0.25 * a.ih2);   // 1/(4h), see cell_slope
    const int os = slot(tx, ty, tz);
    const R tc = LT[os];
    const auto slope = [&](int c, int st, R h) { return cell_slope<R, LIM>(LT[c - st], LT[c], LT[c + st], h); };
    const R sx = slope(os, 1, hih0), sy = slope(os, PX, hih1), sz = slope(os, PP, hih2);
    LS[0][os] = sx;
    LS[1][os] = sy;
    LS[2][os] = sz;
    {
        const bool zr = wave < 2;
        const int hs = zr ? slot(lane % BX, lane / BX, wave == 0 ? -1 : BZ)
                          : slot(lane % BX, wave == 2 ? -1 : BY, lane / BX);
        LS[0][hs] = slope(hs, 1, hih0);
        if (zr) LS[1][hs] = slope(hs, PX, hih1);
        else LS[2][hs] = slope(hs, PP, hih2);
        if (wave == 1 && lane < 2 * BY * BZ) {
            const int c = lane % (BY * BZ), xs = slot(lane < BY * BZ ? -1 : BX, c % BY, c / BY);
            LS[1][xs] = slope(xs, PX, hih1);
            LS[2][xs] = slope(xs, PP, hih2);
        }
    }
    __syncthreads();

    const auto tr = face_transverse<R, LIM>;
    const R fxp = face_flux_dir<R, SAT, KM>(tc, LT[os + 1], ih0, tr(sy, LS[1][os + 1]), tr(sz, LS[2][os + 1]), dx, fk);
    const R fyp = face_flux_dir<R, SAT, KM>(tc, LT[os + PX], ih1, tr(sx, LS[0][os + PX]), tr(sz, LS[2][os + PX]), dy, fk);
    const R fzp = face_flux_dir<R, SAT, KM>(tc, LT[os + PP], ih2, tr(sx, LS[0][os + PP]), tr(sy, LS[1][os + PP]), dz, fk);
    const int ix = (tz * BY + ty) * (BX + 1) + tx, iy = (tz * (BY + 1) + ty) * BX + tx, iz = (tz * BY + ty) * BX + tx;
    FX[ix + 1] = fxp;
    FY[iy + BX] = fyp;
    FZ[iz + BX * BY] = fzp;
    if (job) {
        const int rs = slot(jx, jy, jz), ls = rs - (jobx ? 1 : joby ? PX : PP);
        const R* S1 = jobx ? LS[1] : LS[0];
        const R* S2 = jobz ? LS[1] : LS[2];
        FaceDir<R> dl;
        if (jobx) dl = face_dir(l0, l1, l2, r0, r1, r2);
        else if (joby) dl = face_dir(l1, l0, l2, r1, r0, r2);
        else dl = face_dir(l2, l0, l1, r2, r0, r1);
        const R f = face_flux_dir<R, SAT, KM>(LT[ls], LT[rs], jobx ? ih0 : joby ? ih1 : ih2, tr(S1[ls], S1[rs]),
                                              tr(S2[ls], S2[rs]), dl, fk);
        if (jobx) FX[(jz * BY + jy) * (BX + 1)] = f;
        else if (joby) FY[jz * (BY + 1) * BX + jx] = f;
        else FZ[jy * BX + jx] = f;
    }
    __syncthreads();

    TileExt ex{-INFINITY, INFINITY, 0.0};
    if (store) {
        R div = (fxp - FX[ix]) * ih0;
        div = fma(fyp - FY[iy], ih1, div);
        div = fma(fzp - FZ[iz], ih2, div);
        const double tl = a.scale * (double)div;
        if (a.kind == 0) {
            a.Yout[o] = tl;
        } else if (a.kind == 1) {
            const R m = R(tl);
            ((R*)a.MY0out)[o] = m;
            a.Yout[o] = fma(a.mut, (double)m, yk);
        } else if (a.kind == 3) {
            a.Yout[o] = yk + tl;
        } else {
            const double y = stage_combine(a.mu, a.nu, a.omn, a.mut, a.gt, yk, ym2, yz, tl, (double)my0);
            a.Yout[o] = y;
            ex.mx = fmax(ex.mx, y);
            ex.mn = fmin(ex.mn, y);
            ex.bad = isfinite(y) ? ex.bad : 1.0;
        }
    }
    if (a.ext) store_ext<256>(P, ex);   // uniform: the last stage of a routed sequence
}

template <typename R, bool LIM, int SAT, int KM>
static void block_ask(const StageLaunch& P, int nblocks, hipStream_t st) {
    // routed launches of more than four blocks per CU, and of stages past 64
    if (P.route.A && (nblocks > 1024 || P.stage > 64)) block_kernel<R, LIM, SAT, KM, true><<<nblocks, 256, 0, st>>>(P);
    else block_kernel<R, LIM, SAT, KM, false><<<nblocks, 256, 0, st>>>(P);
}
template <typename R, bool LIM, int KM>
static void block_sat(const StageLaunch& P, int nblocks, int sat, hipStream_t st) {
    if (sat == 2) block_ask<R, LIM, 2, KM>(P, nblocks, st);
    else if (sat == 1) block_ask<R, LIM, 1, KM>(P, nblocks, st);
    else block_ask<R, LIM, 0, KM>(P, nblocks, st);
}
template <typename R, int KM>
static void block_lim(const StageLaunch& P, int nblocks, bool lim, int sat, hipStream_t st) {
    if (lim) block_sat<R, true, KM>(P, nblocks, sat, st);
    else block_sat<R, false, KM>(P, nblocks, sat, st);
}

template <typename R>
hipError_t launch_block(const StageLaunch& P, int nblocks, bool lim, int sat, hipStream_t st) {
    if (P.t.ndim != 3 || P.t.fixed || P.bz != kBlockZ || (int64_t)P.t.n0 * P.t.n1 * P.t.n2 >= (int64_t)1 << 29)
        return hipErrorInvalidValue;   // 32-bit byte offsets
    if (P.kmode == 0) block_lim<R, 0>(P, nblocks, lim, sat, st);
    else if (P.kmode == 1) block_lim<R, 1>(P, nblocks, lim, sat, st);
    else block_lim<R, 2>(P, nblocks, lim, sat, st);
    return hipGetLastError();
}

}  // namespace rkl
