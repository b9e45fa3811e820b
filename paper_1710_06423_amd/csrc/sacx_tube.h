// sacx_tube.h -- a whole RK4 step of a one-dimensional subdomain in one launch
// (ny = 1, y periodic, plain coefficient, no background).
//
// Why: a tube's stage is 4-5 us of latency (launch, load, three barriers) for
// under a microsecond of arithmetic, so a step took 22 us at any length up to
// thousands of cells.  Nothing but the time step is global, and that is fixed
// at the step's start, so a block can take its cells through all four stages
// by itself: it computes 12 more cells on each side (3 per stage) and keeps
// the stage states in registers, sharing primitives and fluxes through LDS.
// 800 points, 40 steps with their initial state and fields read: 0.54 ms
// from 0.92.
//
// A block of NT threads owns NT - 24 cells.  The step reads U and writes the
// new state to another buffer (neighbouring blocks still read U).  Periodic
// images evolve as the cells they image.  At an open end the edge cell's
// thread writes its primitives and fluxes to the three ghost slots beside it
// in every stage, which is what a zero-gradient copy of the stage's input
// gives.
//
// The arithmetic of a stage is that of stage_tile_1d, operation for operation.
#pragma once

#include "sacx_tile.h"

namespace sacx {

template <typename real, int NT, bool HD>
__global__ __launch_bounds__(NT) void k_tube_step(TubeArgs<real> a) {
    __shared__ TubeLds<real, NT> lds;
    constexpr int TX = NT - 8 * G;
    DevScalars *sc = a.sc;
    const Layout L = a.L;
    const int64_t fs = a.fstride;
    const int tid = threadIdx.x;
    const int c = (int)blockIdx.x * TX - 4 * G + tid;
    const bool outcol = tid >= 4 * G && tid < NT - 4 * G && c < L.nx;
    const int64_t oo = (int64_t)L.xoff + c + (int64_t)G * L.pitch;
    if (!sc->active) {
        // stepping ended between the two steps of a pair: the state moves on
        // to the buffer the pair ends in
        if (a.second && sc->prev_active && outcol) {
#pragma unroll
            for (int f = 0; f < NF; ++f) a.out[oo + f * fs] = a.U[oo + f * fs];
        }
        return;
    }
    const real dt = (real)sc->dt, hdt = (real)sc->hdt, dt6 = (real)sc->dt6;
    real kx2[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) kx2[k] = (real)sc->kx2[k];
    const SchemeConsts &kc = a.k;
    const real gamma = (real)kc.gamma, gm1 = (real)kc.gm1, igm1 = (real)kc.igm1;
    const real i12dx = (real)kc.i12dx, idx = (real)kc.idx, i2dx = (real)kc.i2dx, third = (real)kc.third;
    const real half = (real)0.5, two = (real)2, eight = (real)8, zero = (real)0;
    const int tm1 = tid >= 1 ? tid - 1 : 0;
    const int tm2 = tid >= 2 ? tid - 2 : 0;
    const int tp1 = tid + 1 < NT ? tid + 1 : NT - 1;
    const int tp2 = tid + 2 < NT ? tid + 2 : NT - 1;
    const int tp3 = tid + 3 < NT ? tid + 3 : NT - 1;
    auto &sh_fx = lds.fx;
    auto &sh_q = lds.q[0];
    auto &sh_s = lds.s;
    auto &sh_hx = lds.hx;

    // the cell this thread computes: its own, the cell it images, or (past an
    // open end) any cell, unused
    int src = c;
    if (a.periodic) {
        src = c % L.nx;
        src += src < 0 ? L.nx : 0;
    } else {
        src = c < 0 ? 0 : (c >= L.nx ? L.nx - 1 : c);
    }
    // ghost slots of an open end are written by the edge cell's thread
    const bool ghost = !a.periodic && (c < 0 || c >= L.nx);
    const bool edge_lo = a.open_lo && c == 0, edge_hi = a.open_hi && c == L.nx - 1;
    real U[NF], S[NF], A[NF], K[NF];
    {
        const int64_t ro = (int64_t)L.xoff + src + (int64_t)G * L.pitch;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            U[f] = a.U[ro + f * fs];
            S[f] = U[f];
            A[f] = zero;
        }
    }
    double cx_t = 0.0, cy_t = 0.0;
    int bad_t = 0;

#pragma unroll
    for (int stage = 1; stage <= 4; ++stage) {
        const real rt = S[0], mx = S[1], my = S[2], et = S[3], bxt = S[4], byt = S[5];
        const real rho = zero + rt;
        const real irho = recip_t<real, true>(rho);
        const real vx = mx * irho, vy = my * irho;
        const real kin = half * (mx * vx + my * vy);
        const real bbdot = zero * bxt + zero * byt;
        const real bt2 = bxt * bxt + byt * byt;
        const real pk = gm1 * (((et - kin) - bbdot) - half * bt2);
        const real pt = (pk + half * bt2) + bbdot;
        const real eps = pk * igm1;
        const real bxT = zero + bxt, byT = zero + byt;
        const real bvt = bxt * vx + byt * vy;
        const real bvb = zero * vx + zero * vy;
        const real ef = et + zero + pt;
        real fx[5], q[NQ];
        fx[CR] = mx;
        fx[CMX] = (vx * mx - (bxt * bxt + two * bxt * zero)) + pt;
        fx[CMY] = vx * my - (bxt * byt + bxt * zero + zero * byt);
        fx[CE] = ((vx * ef - bxt * bvt) - bxt * bvb) - zero * bvt;
        fx[CB] = vx * byT - bxT * vy;
        q[QR] = rt;
        q[QE] = eps;
        q[QVX] = vx;
        q[QVY] = vy;
        q[QB] = byt;
        q[QRHO] = rho;
        q[QBYT] = byT;
        if (!ghost) {
#pragma unroll
            for (int m = 0; m < 5; ++m) sh_fx[m][tid] = fx[m];
#pragma unroll
            for (int m = 0; m < NQ; ++m) sh_q[m][tid] = q[m];
        }
        if (edge_lo || edge_hi) {
#pragma unroll
            for (int g = 1; g <= G; ++g) {
                const int lo = tid - g, hi = tid + g;
                if (edge_lo && lo >= 0) {
#pragma unroll
                    for (int m = 0; m < 5; ++m) sh_fx[m][lo] = fx[m];
#pragma unroll
                    for (int m = 0; m < NQ; ++m) sh_q[m][lo] = q[m];
                }
                if (edge_hi && hi < NT) {
#pragma unroll
                    for (int m = 0; m < 5; ++m) sh_fx[m][hi] = fx[m];
#pragma unroll
                    for (int m = 0; m < NQ; ++m) sh_q[m][hi] = q[m];
                }
            }
        }
        __syncthreads();
        {
            real dxn[5];
#pragma unroll
            for (int k = 0; k < 5; ++k)
                dxn[k] = (eight * (sh_fx[k][tp1] - sh_fx[k][tm1]) - (sh_fx[k][tp2] - sh_fx[k][tm2])) * i12dx;
            // D_y of any flux is an exact +0 (identical rows)
            K[0] = -(dxn[CR] + zero);
            K[1] = -(dxn[CMX] + zero);
            K[2] = -(dxn[CMY] + zero);
            K[3] = -(dxn[CE] + zero);
            K[4] = -(zero + zero);
            K[5] = -(dxn[CB] + zero);
            if (kc.grav) {
                // gravity on the perturbation density
                const real gx = (real)kc.gx, gy = (real)kc.gy;
                K[1] = K[1] + rt * gx;
                K[2] = K[2] + rt * gy;
                K[3] = K[3] + rt * (gx * vx + gy * vy);
            }
        }
        if (HD) {
            const real dv = (sh_q[QVX][tp1] - sh_q[QVX][tm1]) * i2dx + zero;
            const real s_c = fmax(zero, -dv);
            sh_s[tid] = s_c;
            __syncthreads();
            const real sfx = fmax(s_c, sh_s[tp1]);
            real gx[5];
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const int cl = qclass(k);
                const real q0 = sh_q[k][tm2], q1 = sh_q[k][tm1], q2 = sh_q[k][tid];
                const real q3 = sh_q[k][tp1], q4 = sh_q[k][tp2], q5 = sh_q[k][tp3];
                const real R = hd_ratio_t<real, true>(q0, q1, q2, q3, q4, q5);
                const real nu = kx2[cl] * R + (real)kc.kxs[cl] * sfx;
                gx[k] = nu * (q3 - q2) * idx;
            }
            const real rf = half * (sh_q[QRHO][tid] + sh_q[QRHO][tp1]);
            const real vxf = half * (sh_q[QVX][tid] + sh_q[QVX][tp1]);
            const real vyf = half * (sh_q[QVY][tid] + sh_q[QVY][tp1]);
            const real byf = half * (sh_q[QBYT][tid] + sh_q[QBYT][tp1]);
            // the four-face averages of y-face G vanish exactly (G_y = +0)
            const real txx = rf * gx[QVX];
            const real txy = half * rf * (gx[QVY] + zero);
            const real ez = gx[QB] - zero;
            sh_hx[CR][tid] = gx[QR];
            sh_hx[CMX][tid] = txx;
            sh_hx[CMY][tid] = txy;
            sh_hx[CE][tid] = (gx[QE] + (vxf * txx + vyf * txy)) + byf * ez;
            sh_hx[CB][tid] = ez;
            __syncthreads();
            // H_y is the same on both y faces of the row: its difference is +0
            K[0] = K[0] + ((sh_hx[CR][tid] - sh_hx[CR][tm1]) * idx + zero);
            K[1] = K[1] + ((sh_hx[CMX][tid] - sh_hx[CMX][tm1]) * idx + zero);
            K[2] = K[2] + ((sh_hx[CMY][tid] - sh_hx[CMY][tm1]) * idx + zero);
            K[3] = K[3] + ((sh_hx[CE][tid] - sh_hx[CE][tm1]) * idx + zero);
            K[4] = K[4] + (zero + zero);
            K[5] = K[5] + ((sh_hx[CB][tid] - sh_hx[CB][tm1]) * idx + zero);
        } else {
            __syncthreads();   // the fluxes have been read
        }
        if (stage == 1) {
#pragma unroll
            for (int f = 0; f < NF; ++f) S[f] = S[f] + hdt * K[f];
        } else if (stage == 2) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const real u = U[f], s = S[f];
                S[f] = u + hdt * K[f];
                A[f] = (u + u) + ((s - u) + dt * K[f]);
            }
        } else if (stage == 3) {
#pragma unroll
            for (int f = 0; f < NF; ++f) S[f] = U[f] + dt * K[f];
        } else if (outcol) {
            real un[6];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const real av = A[f], s = S[f];
                un[f] = (s + (av - (s + s)) * third) + dt6 * K[f];
                a.out[oo + f * fs] = un[f];
            }
            const real r0 = zero + un[0];
            const real ir0 = (real)1 / r0;
            const real ux = un[1] * ir0, uy = un[2] * ir0;
            const real kn = half * (un[1] * ux + un[2] * uy);
            const real bbd = zero * un[4] + zero * un[5];
            const real b2t = un[4] * un[4] + un[5] * un[5];
            const real pkt = gm1 * (((un[3] - kn) - bbd) - half * b2t);
            const real b2b = zero * zero + zero * zero;
            const real pkb = gm1 * (zero - half * b2b);
            const real pkk = pkb + pkt;
            const real bxx = zero + un[4], byy = zero + un[5];
            const real cf = sqrt((gamma * pkk + (bxx * bxx + byy * byy)) * ir0);
            const bool fin = isfinite(un[0]) && isfinite(un[1]) && isfinite(un[2]) && isfinite(un[3]) &&
                             isfinite(un[4]) && isfinite(un[5]) && isfinite(cf);
            if (!(r0 > (real)0) || !(pkk > (real)0) || !fin) {
                bad_t = 1;
            } else {
                cx_t = fmax(cx_t, (double)(fabs(ux) + cf));
                cy_t = fmax(cy_t, (double)(fabs(uy) + cf));
            }
        }
    }
    raise_speeds(cx_t, cy_t, bad_t, lds.red, sc, sc->cur ^ 1);
}

template <typename real, int NT>
static hipError_t launch_tube_nt(bool hd, const TubeArgs<real> &a, hipStream_t s) {
    constexpr int TX = NT - 8 * G;
    const dim3 g((a.L.nx + TX - 1) / TX);
    if (hd) hipLaunchKernelGGL((k_tube_step<real, NT, true>), g, dim3(NT), 0, s, a);
    else hipLaunchKernelGGL((k_tube_step<real, NT, false>), g, dim3(NT), 0, s, a);
    return hipGetLastError();
}

// One wave per block (40 of its 64 cells written, no wait for other waves)
// while that makes at most a block per compute unit (of 256): 800 cells 14.7 ->
// 13.4 us per step in FP64 and 12.5 -> 11.6 in FP32, 3000 15.4 -> 13.3 and
// 12.9 -> 11.7.  Longer tubes recompute less with four: 200000 cells 38 us and
// 27 us, against 42 and 33.
template <typename real>
hipError_t launch_tube_step(bool hd, int cus, const TubeArgs<real> &a, hipStream_t s) {
    return a.L.nx <= (int64_t)cus * (64 - 8 * G) ? launch_tube_nt<real, 64>(hd, a, s) : launch_tube_nt<real, 256>(hd, a, s);
}

}  // namespace sacx
