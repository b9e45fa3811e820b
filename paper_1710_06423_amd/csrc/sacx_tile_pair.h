// sacx_tile_pair.h -- two RK stages of the scheme without hyper-diffusion in
// one launch (two-dimensional subdomains, no background).
//
// Why: without hyper-diffusion a stage is bound by memory.  1501 x 997 in FP64
// moves 144 to 288 MB a launch, and the four launches ran at 3.6-5.0 TB/s,
// where a large copy reaches 4.7.  A stage reads only two cells to each side,
// so a block can take its cells through two stages by itself: stages 1 and 2
// read U and write w2 and A, stages 3 and 4 read w2, U and A and write the new
// state.  Seven passes over the fields per step instead of twelve.
//
// Block: W waves over 64 columns (56 written) and W*R rows (W*R - 8 written),
// a wave holding R neighbouring rows, a lane per column.  D_x F_x goes through
// register lanes, the y fluxes through LDS.  The first stage's result stays in
// registers: valid two cells inside the loaded box, of which the second stage
// is valid four cells inside.  Beyond an open side the first stage's result is
// that of the edge cell, as a stage launch would read it: across x from the
// edge's lane, across y through LDS.  Periodic images evolve as their cells.
//
// The new state goes to another buffer than U, which neighbouring blocks still
// read; steps are taken in twos, so that a call ends with its state in U.
//
// The arithmetic is that of the stage kernels, operation for operation.
//
// Measured, us per step, one stage per launch: FP64 300 x 136 30.0, 900 x 700
// 105, 1501 x 997 197, 4000^2 2524; FP32 300 x 136 24.5, 1501 x 997 114, 4000^2
// 1069.  This with 8 and with 24 rows written per block: FP64 19.0, 26.6; 68, 67;
// 148, 150; 1493, 1369.  FP32 16.3, 18.8; 78, 76; 808, 728.  Three rows per wave
// took 128 registers and 100-156 B of scratch in FP64 (4000^2: 1928).
#pragma once

#include "sacx_tile_box.h"

namespace sacx {

template <typename real, int W, int R>
struct PairLds {
    real fy[5][W * R][64];
    real edge[2][NF][64];   // first-stage result of the cells at the open ends of y
    double red[3][W];
};

// the value of one lane, the same in all
__device__ __forceinline__ float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// where cell i of a direction of n cells is read: its periodic image, or the
// edge cell beyond an open side; cells more than 4 outside are read
// somewhere, unused
__device__ __forceinline__ int pair_cell(const SideMap &m, int i) {
    int j = i;
    if (m.below) j = i < 0 ? i + m.n : (i >= m.n ? i - m.n : i);
    return j < 0 ? 0 : (j >= m.n ? m.n - 1 : j);
}

// LAST: stages 3 and 4, otherwise 1 and 2
template <typename real, int W, int R, bool LAST>
__device__ __forceinline__ void stage_tile_pair(const StageArgs<real> &a, bool second, int tile_x, int tile_y,
                                                PairLds<real, W, R> &lds) {
    constexpr int TX = 56, NB = W * R, TY = NB - 8;
    const Layout L = a.L;
    const int64_t fs = a.fstride;
    const int t = (int)threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = tile_x * TX - 4 + t, y0 = tile_y * TY, i0 = w * R;   // box row i is row y0 - 4 + i
    const bool outcol = t >= 4 && t < 60 && c < L.nx;
    const DevScalars *sc = a.sc;
    if (!sc->active) {
        // stepping ended between the two steps of a pair: the state moves on
        // to the buffer the pair ends in
        if (LAST && second && sc->prev_active) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int i = i0 + k, y = y0 - 4 + i;
                if (i < 4 || i >= NB - 4 || y >= L.ny || !outcol) continue;
                const int64_t o = (int64_t)L.xoff + c + (int64_t)(y + G) * L.pitch;
#pragma unroll
                for (int f = 0; f < NF; ++f) a.out1[0][o + f * fs] = a.U[0][o + f * fs];
            }
        }
        return;
    }
    const real dt = (real)sc->dt, hdt = (real)sc->hdt, dt6 = (real)sc->dt6;
    const SchemeConsts &kc = a.k;
    const real gamma = (real)kc.gamma, gm1 = (real)kc.gm1, third = (real)kc.third;
    const real i12dx = (real)kc.i12dx, i12dy = (real)kc.i12dy;
    const real half = (real)0.5, two = (real)2, eight = (real)8, zero = (real)0;

    const int64_t co = (int64_t)L.xoff + pair_cell(a.mx, c);
    auto src = [&](int k) -> int64_t {
        return co + (int64_t)(pair_cell(a.my, y0 - 4 + i0 + k) + G) * L.pitch;
    };
    Row6<real> s[R], p[R];   // the stage's input; the combine's stored operand
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t o = src(k);
#pragma unroll
        for (int f = 0; f < NF; ++f) s[k].v[f] = a.S[0][o + f * fs];
    }
    if (LAST) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int64_t o = src(k);
#pragma unroll
            for (int f = 0; f < NF; ++f) p[k].v[f] = a.U[0][o + f * fs];
        }
    }

    // -(D_x F_x + D_y F_y) of the wave's rows from their states s, valid for
    // rows and lanes with two valid neighbours to each side
    real K[R][6];
    auto ideal = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const real rt = s[k].v[0], mx = s[k].v[1], my = s[k].v[2], et = s[k].v[3], bxt = s[k].v[4],
                       byt = s[k].v[5];
            const real rb = 0, eb = 0, bxb = 0, byb = 0;
            const real rho = rb + rt;
            const real irho = recip_t<real, true>(rho);
            const real vx = mx * irho, vy = my * irho;
            const real kin = half * (mx * vx + my * vy);
            const real bbdot = bxb * bxt + byb * byt;
            const real bt2 = bxt * bxt + byt * byt;
            const real pk = gm1 * (((et - kin) - bbdot) - half * bt2);
            const real pt = (pk + half * bt2) + bbdot;
            const real bxT = bxb + bxt, byT = byb + byt;
            const real bvt = bxt * vx + byt * vy;
            const real bvb = bxb * vx + byb * vy;
            const real ef = et + eb + pt;
            real fx[5], fy[5];
            fx[CR] = mx;
            fx[CMX] = (vx * mx - (bxt * bxt + two * bxt * bxb)) + pt;
            fx[CMY] = vx * my - (bxt * byt + bxt * byb + bxb * byt);
            fx[CE] = ((vx * ef - bxt * bvt) - bxt * bvb) - bxb * bvt;
            fx[CB] = vx * byT - bxT * vy;
            fy[CR] = my;
            fy[CMX] = vy * mx - (byt * bxt + byt * bxb + byb * bxt);
            fy[CMY] = (vy * my - (byt * byt + two * byt * byb)) + pt;
            fy[CE] = ((vy * ef - byt * bvt) - byt * bvb) - byb * bvt;
            fy[CB] = vy * bxT - byT * vx;
#pragma unroll
            for (int m = 0; m < 5; ++m) {
                lds.fy[m][i0 + k][t] = fy[m];
                const real l1 = lane_left(fx[m]), l2 = lane_left(l1), r1 = lane_right(fx[m]), r2 = lane_right(r1);
                K[k][m < CB ? m : 5] = (eight * (r1 - l1) - (r2 - l2)) * i12dx;
                settle(K[k][m < CB ? m : 5]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 5; ++m) {
            // rows i0-2 .. i0+R+1, clamped into the box (unused there)
            real fw[R + 4];
#pragma unroll
            for (int k = 0; k < R + 4; ++k) fw[k] = lds.fy[m][min(max(i0 + k - 2, 0), NB - 1)][t];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const real dy = (eight * (fw[k + 3] - fw[k + 1]) - (fw[k + 4] - fw[k])) * i12dy;
                if (m < CB) {
                    K[k][m] = -(K[k][m] + dy);
                    settle(K[k][m]);
                } else {
                    K[k][4] = -(zero + dy);        // B~_x has no x flux
                    K[k][5] = -(K[k][5] + zero);   // B~_y has no y flux
                    settle(K[k][4]);
                    settle(K[k][5]);
                }
            }
        }
        if (kc.grav) {
            const real gx = (real)kc.gx, gy = (real)kc.gy;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const real rg = s[k].v[0];
                const real irho = recip_t<real, true>(zero + rg);
                const real vx = s[k].v[1] * irho, vy = s[k].v[2] * irho;
                K[k][1] = K[k][1] + rg * gx;
                K[k][2] = K[k][2] + rg * gy;
                K[k][3] = K[k][3] + rg * (gx * vx + gy * vy);
            }
        }
    };

    // ---- the first of the two stages, its result in s
    ideal();
#pragma unroll
    for (int k = 0; k < R; ++k) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (LAST) s[k].v[f] = p[k].v[f] + dt * K[k][f];
            else s[k].v[f] = s[k].v[f] + hdt * K[k][f];
            settle(s[k].v[f]);
        }
    }
    // cells beyond an open side (sides are tested for the whole block)
    const int xl = 4, xh = L.nx - 1 - tile_x * TX + 4;   // lanes of the first and last column
    const bool fxl = a.mx.lo == 0 && tile_x == 0, fxh = a.mx.hi == L.nx - 1 && xh < 63;
    if (fxl || fxh) {
#pragma unroll
        for (int k = 0; k < R; ++k)
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                real v = s[k].v[f];
                if (fxl) { const real e = lane_value(v, xl); v = t < xl ? e : v; }
                if (fxh) { const real e = lane_value(v, xh); v = t > xh ? e : v; }
                s[k].v[f] = v;
            }
    }
    const int yl = 4, yh = L.ny - 1 - y0 + 4;            // box rows of the first and last row
    const bool fyl = a.my.lo == 0 && tile_y == 0, fyh = a.my.hi == L.ny - 1 && yh < NB - 1;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int i = i0 + k;
        if (fyl && i == yl) {
#pragma unroll
            for (int f = 0; f < NF; ++f) lds.edge[0][f][t] = s[k].v[f];
        }
        if (fyh && i == yh) {
#pragma unroll
            for (int f = 0; f < NF; ++f) lds.edge[1][f][t] = s[k].v[f];
        }
    }
    // the second stage's stored operand: U, or A at stage 4
    int64_t oo[R];
    bool outrow[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int i = i0 + k, y = y0 - 4 + i;
        outrow[k] = outcol && i >= 4 && i < NB - 4 && y < L.ny;
        oo[k] = (int64_t)L.xoff + c + (int64_t)(y + G) * L.pitch;
        if (outrow[k]) {
#pragma unroll
            for (int f = 0; f < NF; ++f) p[k].v[f] = (LAST ? a.A[0] : a.U[0])[oo[k] + f * fs];
        }
    }
    __syncthreads();   // the y fluxes have been read, the edge rows written
    if (fyl || fyh) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int i = i0 + k;
            if (fyl && i < yl) {
#pragma unroll
                for (int f = 0; f < NF; ++f) s[k].v[f] = lds.edge[0][f][t];
            }
            if (fyh && i > yh) {
#pragma unroll
                for (int f = 0; f < NF; ++f) s[k].v[f] = lds.edge[1][f][t];
            }
        }
    }

    // ---- the second
    ideal();
    double cx_t = 0.0, cy_t = 0.0;
    int bad_t = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if (!outrow[k]) continue;
        const int64_t o = oo[k];
        if (!LAST) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const real uv = p[k].v[f], sv = s[k].v[f];
                a.out1[0][o + f * fs] = uv + hdt * K[k][f];
                a.out2[0][o + f * fs] = (uv + uv) + ((sv - uv) + dt * K[k][f]);
            }
        } else {
            real un[6];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const real av = p[k].v[f], sv = s[k].v[f];
                un[f] = (sv + (av - (sv + sv)) * third) + dt6 * K[k][f];
                a.out1[0][o + f * fs] = un[f];
            }
            const real rb0 = 0, eb0 = 0, bxb0 = 0, byb0 = 0;
            const real r0 = rb0 + un[0];
            const real ir0 = (real)1 / r0;
            const real ux = un[1] * ir0, uy = un[2] * ir0;
            const real kn = half * (un[1] * ux + un[2] * uy);
            const real bbd = bxb0 * un[4] + byb0 * un[5];
            const real b2t = un[4] * un[4] + un[5] * un[5];
            const real pkt = gm1 * (((un[3] - kn) - bbd) - half * b2t);
            const real b2b = bxb0 * bxb0 + byb0 * byb0;
            const real pkb = gm1 * (eb0 - half * b2b);
            const real pkk = pkb + pkt;
            const real bxx = bxb0 + un[4], byy = byb0 + un[5];
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
    if (LAST) raise_speeds(cx_t, cy_t, bad_t, lds.red, a.sc, a.sc->cur ^ 1);
}

template <typename real, int W, int R, bool LAST>
__global__ __launch_bounds__(64 * W, 4) void k_stage_pair(StageArgs<real> a, int second) {
    __shared__ PairLds<real, W, R> lds;
    int tx, ty;
    xcd_tile<4>(tx, ty);
    stage_tile_pair<real, W, R, LAST>(a, second != 0, tx, ty, lds);
}

template <typename real, int W>
static hipError_t launch_pair_w(bool last, bool second, const StageArgs<real> &a, hipStream_t s) {
    constexpr int R = 2, TY = W * R - 8;
    const dim3 g((a.L.nx + 55) / 56, (a.L.ny + TY - 1) / TY), t(64 * W);
    if (last) hipLaunchKernelGGL((k_stage_pair<real, W, R, true>), g, t, 0, s, a, second);
    else hipLaunchKernelGGL((k_stage_pair<real, W, R, false>), g, t, 0, s, a, second);
    return hipGetLastError();
}

// rows: 8 or 24 per block
template <typename real>
hipError_t launch_pair(bool last, bool second, int rows, const StageArgs<real> &a, hipStream_t s) {
    return rows == 24 ? launch_pair_w<real, 16>(last, second, a, s) : launch_pair_w<real, 8>(last, second, a, s);
}

}  // namespace sacx
