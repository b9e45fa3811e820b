// sacx_tile_box.h -- the fused RK stage on a box of cells held in LDS (plain
// coefficient, no background), for grids whose strips would be short.
//
// Why: the marching tiles take a block about 1.5-2.7 us per row, a latency
// (three barriers and their LDS round trips in series), and 6 warm-up rows per
// strip; where a grid has few rows per strip that latency is the launch's
// time.  Here the rows of a block run side by side, a wave for each R of them,
// so a stage is four barriers whatever the grid: 7-8 us for one block per
// compute unit in FP64.  Per step, against the best marching shape: 300 x 136
// 41 us from 77, 512^2 88 from 137, 1024^2 206 from 261, 2048^2 827 from 796
// (FP64); 31 from 72, 55 from 97, 115 from 158, 368 from 395 (FP32).  What
// bounds it at size is the apron (14 rows loaded for 8, about 1.9 times the
// primitives) and LDS traffic (about 170 reads and writes per cell).
//
// Block: W waves, wave w the R output rows y0 + wR .., lane t the column
// x0 - 3 + t (58 output columns, the 3-cell apron on each side computed by the
// edge lanes).  Rows are numbered from the first output row; the box holds
// rows -3 .. TY+2, TY = W R.
//   P1  state, primitives and fluxes of the own rows and of the apron rows
//       dealt to the wave; x and y fluxes and the velocities to LDS
//   P2  D_x F_x, D_y F_y and the ideal L of the own rows; compression s
//   P3  (rho~, eps~, B~ to LDS, over the fluxes) face G: the own rows' x
//       faces and upper y faces; one wave each also the y faces below the
//       box and the x faces (v_y, B_y) of the rows below and above it
//   P4  face fluxes, L(S), the stage combine, in stage 4 the wave speeds
// Every value is the same operation on the same operands as in the marching
// tiles, so all give the same bits.
//
// LDS: 80 KB in FP64 with eight rows (the fluxes and what follows them share
// memory), so that two blocks of eight waves, four waves per SIMD, share a
// compute unit.
#pragma once

#include "sacx_tile.h"

namespace sacx {

template <typename real, int W, int R, bool HD>
struct BoxLds {
    static constexpr int TY = W * R, NB = TY + 6;
    struct Flux {
        real fx[5][TY][64];       // x fluxes of rows 0 .. TY-1
        real fy[5][TY + 4][64];   // y fluxes of rows -2 .. TY+1
    };
    struct Face {
        real q[4][NB][64];        // rho~, eps~, B~_x, B~_y of rows -3 .. TY+2
        real gx[2][TY + 2][64];   // x-face G(v_y), G(B~_y) of rows -1 .. TY
        real gy[2][TY + 1][64];   // y-face G(v_x), G(B~_x) of faces -1/2 .. TY-1/2
        real gb[3][W + 1][64];    // y-face G(rho~), G(eps~), G(v_y) below each wave's first row
    };
    union {
        Flux f;
        Face g[1];
    };
    real v[2][HD ? NB : 1][64];   // v_x, v_y of rows -3 .. TY+2
    real s[HD ? TY + 2 : 1][64];  // compression of rows -1 .. TY
    double red[3][W];
};

// the value of the lane to the left (lane 0 keeps its own, unused)
__device__ __forceinline__ float lane_left(float v) {
    const int i = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ double lane_left(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xf, 0xf, false));
}

// the value of the lane to the right (lane 63 keeps its own, unused)
__device__ __forceinline__ float lane_right(float v) {
    const int i = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ double lane_right(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x130, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(lo, lo, 0x130, 0xf, 0xf, false));
}

// computes v here: the compiler would otherwise sink the arithmetic into the
// block that uses it, up to four barriers later, and hold all its operands
// instead
template <typename real>
__device__ __forceinline__ void settle(real &v) {
    asm volatile("" : "+v"(v));
}

template <typename real, int W, int R, int STAGE, bool HD>
__device__ __forceinline__ void stage_tile_box(const StageArgs<real> &a, int tile_x, int tile_y,
                                               BoxLds<real, W, R, HD> &lds) {
    // rows a wave loads: its own and 1 (W = 8) or up to 2 (W = 4) of the apron's 6
    constexpr int TX = 64 - 2 * G, TY = W * R, NA = W >= 6 ? 1 : 2, NK = R + NA;
    // the waves that take the y faces below the box and the x faces of the
    // rows below and above it (those with the fewest apron rows)
    constexpr int WB = W - 1, WL = W - 2, WH = W - 3;
    const DevScalars *sc = a.sc;
    if (!sc->active) return;
    const real dt = (real)sc->dt, hdt = (real)sc->hdt, dt6 = (real)sc->dt6;
    // (read before the first store, so that they stay scalar)
    real kx2[4], ky2[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) { kx2[k] = (real)sc->kx2[k]; ky2[k] = (real)sc->ky2[k]; }
    const SchemeConsts &kc = a.k;
    const real gamma = (real)kc.gamma, gm1 = (real)kc.gm1, igm1 = (real)kc.igm1;
    const real i12dx = (real)kc.i12dx, i12dy = (real)kc.i12dy, idx = (real)kc.idx, idy = (real)kc.idy;
    const real i2dx = (real)kc.i2dx, i2dy = (real)kc.i2dy, third = (real)kc.third;
    const real half = (real)0.5, two = (real)2, eight = (real)8, zero = (real)0;
    const Layout L = a.L;
    const int64_t fs = a.fstride;
    const int t = (int)threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = tile_x * TX - G + t;
    const int y0 = tile_y * TY;
    const int tm1 = t >= 1 ? t - 1 : 0, tm2 = t >= 2 ? t - 2 : 0;
    const int tp1 = t < 63 ? t + 1 : 63, tp2 = t < 62 ? t + 2 : 63, tp3 = t < 61 ? t + 3 : 63;
    const bool outcol = t >= G && t < 64 - G && c < L.nx;
    const int64_t colofs = (int64_t)L.xoff + a.mx.at(min(c, L.nx + G - 1));
    const int j0 = w * R;   // first own row

    // ================= P1 =================
    // the rows of this wave: its own, then apron rows (-3, -2, -1, TY, TY+1,
    // TY+2 dealt to the waves in turn)
    int row[NK];
    bool has[NK];
#pragma unroll
    for (int k = 0; k < R; ++k) { row[k] = j0 + k; has[k] = true; }
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        const int i = w + k * W;
        has[R + k] = i < 6;
        row[R + k] = i < 3 ? i - 3 : TY + i - 3;
    }
    Row6<real> u[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        if (!has[k]) continue;
        // rows and columns past the last ghost repeat it, unused
        const int64_t o = colofs + (int64_t)(a.my.at(min(y0 + row[k], L.ny + G - 1)) + G) * L.pitch;
#pragma unroll
        for (int f = 0; f < NF; ++f) u[k].v[f] = a.S[0][o + f * fs];
    }
    real vx[NK], vy[NK], eps[NK], fyo[R][5];
    // D_x F_x through register lanes in FP64, where LDS is as busy as the
    // vector units (2 x 2 subdomains of 1024^2 in all 1291 -> 1268 us, 1024^2
    // 2104 -> 2092); FP32 is bound by vector issue (2048^2 3700 -> 3715 us,
    // 8 tubes and 8 boxes 2934 -> 3014) and goes through LDS
    constexpr bool LANES = sizeof(real) == 8;
    real dxo[R][5];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        if (!has[k]) continue;
        const real rt = u[k].v[0], mx = u[k].v[1], my = u[k].v[2], et = u[k].v[3], bxt = u[k].v[4], byt = u[k].v[5];
        const real rb = 0, eb = 0, bxb = 0, byb = 0;
        const real rho = rb + rt;
        const real irho = recip_t<real, true>(rho);
        vx[k] = mx * irho;
        vy[k] = my * irho;
        const real kin = half * (mx * vx[k] + my * vy[k]);
        const real bbdot = bxb * bxt + byb * byt;
        const real bt2 = bxt * bxt + byt * byt;
        const real pk = gm1 * (((et - kin) - bbdot) - half * bt2);
        const real pt = (pk + half * bt2) + bbdot;
        eps[k] = pk * igm1;
        settle(eps[k]);
        const real bxT = bxb + bxt, byT = byb + byt;
        const real bvt = bxt * vx[k] + byt * vy[k];
        const real bvb = bxb * vx[k] + byb * vy[k];
        const real ef = et + eb + pt;
        if (HD) {
            lds.v[0][row[k] + 3][t] = vx[k];
            lds.v[1][row[k] + 3][t] = vy[k];
        }
        if (k < R) {
            real fx[5];
            fx[CR] = mx;
            fx[CMX] = (vx[k] * mx - (bxt * bxt + two * bxt * bxb)) + pt;
            fx[CMY] = vx[k] * my - (bxt * byt + bxt * byb + bxb * byt);
            fx[CE] = ((vx[k] * ef - bxt * bvt) - bxt * bvb) - bxb * bvt;
            fx[CB] = vx[k] * byT - bxT * vy[k];
#pragma unroll
            for (int m = 0; m < 5; ++m) {
                if constexpr (LANES) {
                    const real l1 = lane_left(fx[m]), l2 = lane_left(l1), r1 = lane_right(fx[m]), r2 = lane_right(r1);
                    dxo[k][m] = (eight * (r1 - l1) - (r2 - l2)) * i12dx;
                    settle(dxo[k][m]);
                } else {
                    lds.f.fx[m][row[k]][t] = fx[m];
                }
            }
        }
        if (k < R || (row[k] >= -2 && row[k] <= TY + 1)) {
            real fy[5];
            fy[CR] = my;
            fy[CMX] = vy[k] * mx - (byt * bxt + byt * bxb + byb * bxt);
            fy[CMY] = (vy[k] * my - (byt * byt + two * byt * byb)) + pt;
            fy[CE] = ((vy[k] * ef - byt * bvt) - byt * bvb) - byb * bvt;
            fy[CB] = vy[k] * bxT - byT * vx[k];
#pragma unroll
            for (int m = 0; m < 5; ++m) {
                lds.f.fy[m][row[k] + 2][t] = fy[m];
                if (k < R) fyo[k][m] = fy[m];
            }
        }
    }
    __syncthreads();

    // ================= P2 =================
    real K[R][6];
    {
        // y fluxes of rows j0-2 .. j0+R+1 of the own column
#pragma unroll
        for (int m = 0; m < 5; ++m) {
            real fw[R + 4];
#pragma unroll
            for (int k = 0; k < R + 4; ++k) fw[k] = k >= 2 && k < R + 2 ? fyo[k - 2][m] : lds.f.fy[m][j0 + k][t];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const real dy = (eight * (fw[k + 3] - fw[k + 1]) - (fw[k + 4] - fw[k])) * i12dy;
                real dx;
                if constexpr (LANES) {
                    dx = dxo[k][m];
                } else {
                    const real *fx = lds.f.fx[m][j0 + k];
                    dx = (eight * (fx[tp1] - fx[tm1]) - (fx[tp2] - fx[tm2])) * i12dx;
                }
                if (m < CB) {
                    K[k][m] = -(dx + dy);
                    settle(K[k][m]);
                } else {
                    K[k][4] = -(zero + dy);   // B~_x has no x flux
                    K[k][5] = -(dx + zero);   // B~_y has no y flux
                    settle(K[k][4]);
                    settle(K[k][5]);
                }
            }
        }
    }
    if (kc.grav) {
        const real gx = (real)kc.gx, gy = (real)kc.gy;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const real rg = u[k].v[0];
            K[k][1] = K[k][1] + rg * gx;
            K[k][2] = K[k][2] + rg * gy;
            K[k][3] = K[k][3] + rg * (gx * vx[k] + gy * vy[k]);
        }
    }
    // the combine's stored operand, for the end of the stage
    Row6<real> pU[R];
    bool outrow[R];
    int64_t oo[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        outrow[k] = outcol && y0 + j0 + k < L.ny;
        oo[k] = (int64_t)L.xoff + c + (int64_t)(y0 + j0 + k + G) * L.pitch;
        if (outrow[k] && STAGE > 1) {
#pragma unroll
            for (int f = 0; f < NF; ++f) pU[k].v[f] = (STAGE == 4 ? a.A[0] : a.U[0])[oo[k] + f * fs];
        }
    }
    if constexpr (HD) {
        auto &g = lds.g[0];
        const bool cross = a.hd_cross_on != 0;
        // compression of row j
        auto comp = [&](int j, real vyp, real vym) {
            const real dv = (lds.v[0][j + 3][tp1] - lds.v[0][j + 3][tm1]) * i2dx + (vyp - vym) * i2dy;
            return fmax(zero, -dv);
        };
        real so[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            so[k] = comp(j0 + k, k + 1 < R ? vy[k + 1] : lds.v[1][j0 + k + 4][t],
                         k > 0 ? vy[k - 1] : lds.v[1][j0 + k + 2][t]);
            settle(so[k]);
            lds.s[j0 + k + 1][t] = so[k];
        }
        const int je = w == WL ? -1 : TY;
        real se = zero;
        if (w == WL || w == WH) {
            se = comp(je, lds.v[1][je + 4][t], lds.v[1][je + 2][t]);
            lds.s[je + 1][t] = se;
        }
        __syncthreads();   // the fluxes have been read

        // ================= P3 =================
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            if (!has[k]) continue;
            g.q[0][row[k] + 3][t] = u[k].v[0];
            g.q[1][row[k] + 3][t] = eps[k];
            g.q[2][row[k] + 3][t] = u[k].v[4];
            g.q[3][row[k] + 3][t] = u[k].v[5];
        }
        __syncthreads();
        // a quantity of the x-face set (QB: B~_y) or the y-face set (QB: B~_x) at row j
        auto xrow = [&](int q, int j) -> const real * {
            return q == QR ? g.q[0][j + 3] : (q == QE ? g.q[1][j + 3] : (q == QVX ? lds.v[0][j + 3]
                   : (q == QVY ? lds.v[1][j + 3] : g.q[3][j + 3])));
        };
        auto yat = [&](int q, int j) -> real {
            return q == QR ? g.q[0][j + 3][t] : (q == QE ? g.q[1][j + 3][t] : (q == QVX ? lds.v[0][j + 3][t]
                   : (q == QVY ? lds.v[1][j + 3][t] : g.q[2][j + 3][t])));
        };
        auto own = [&](int q, int k) -> real {
            return q == QR ? u[k].v[0] : (q == QE ? eps[k] : (q == QVX ? vx[k] : (q == QVY ? vy[k] : u[k].v[4])));
        };
        auto xface = [&](int q, int j, real sf) -> real {
            const real *p = xrow(q, j);
            const real q2 = p[t], q3 = p[tp1];
            const real Rt = hd_ratio_t<real, true>(p[tm2], p[tm1], q2, q3, p[tp2], p[tp3]);
            const int cl = qclass(q);
            const real nu = kx2[cl] * Rt + (real)kc.kxs[cl] * sf;
            return nu * (q3 - q2) * idx;
        };
        real gx[R][5];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const real sf = fmax(so[k], lds.s[j0 + k + 1][tp1]);
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                gx[k][q] = xface(q, j0 + k, sf);
                settle(gx[k][q]);
            }
            g.gx[0][j0 + k + 1][t] = gx[k][QVY];
            g.gx[1][j0 + k + 1][t] = gx[k][QB];
        }
        if (w == WL || w == WH) {
            const real sf = fmax(se, lds.s[je + 1][tp1]);
            g.gx[0][je + 1][t] = xface(QVY, je, sf);
            g.gx[1][je + 1][t] = xface(QB, je, sf);
        }
        // upper y faces of the own rows (face k above row j0+k)
        real gy[R][5];
        const real sup = lds.s[j0 + R + 1][t];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            real qw[R + 5];   // rows j0-2 .. j0+R+2
#pragma unroll
            for (int k = 0; k < R + 5; ++k) qw[k] = k >= 2 && k < R + 2 ? own(q, k - 2) : yat(q, j0 - 2 + k);
            const int cl = qclass(q);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const real sf = fmax(so[k], k + 1 < R ? so[k + 1 < R ? k + 1 : k] : sup);
                const real Rt = hd_ratio_t<real, true>(qw[k], qw[k + 1], qw[k + 2], qw[k + 3], qw[k + 4], qw[k + 5]);
                const real nu = ky2[cl] * Rt + (real)kc.kys[cl] * sf;
                gy[k][q] = nu * (qw[k + 3] - qw[k + 2]) * idy;
                settle(gy[k][q]);
            }
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            g.gy[0][j0 + k + 1][t] = gy[k][QVX];
            g.gy[1][j0 + k + 1][t] = gy[k][QB];
        }
        g.gb[0][w + 1][t] = gy[R - 1][QR];
        g.gb[1][w + 1][t] = gy[R - 1][QE];
        g.gb[2][w + 1][t] = gy[R - 1][QVY];
        if (w == WB) {
            // the face below the box (row -1 to row 0)
            const real sf = fmax(lds.s[0][t], lds.s[1][t]);
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const int cl = qclass(q);
                const real q2 = yat(q, -1), q3 = yat(q, 0);
                const real Rt = hd_ratio_t<real, true>(yat(q, -3), yat(q, -2), q2, q3, yat(q, 1), yat(q, 2));
                const real nu = ky2[cl] * Rt + (real)kc.kys[cl] * sf;
                const real gq = nu * (q3 - q2) * idy;
                if (q == QVX) g.gy[0][0][t] = gq;
                else if (q == QB) g.gy[1][0][t] = gq;
                else g.gb[q == QR ? 0 : (q == QE ? 1 : 2)][0][t] = gq;
            }
        }
        __syncthreads();

        // ================= P4 =================
        // G on the face below the first own row
        real gbot[5];
        gbot[QR] = g.gb[0][w][t];
        gbot[QE] = g.gb[1][w][t];
        gbot[QVY] = g.gb[2][w][t];
        gbot[QVX] = g.gy[0][j0][t];
        gbot[QB] = g.gy[1][j0][t];
        // H_y on the face between rows m and m+1 of the own column
        auto yflux = [&](int m, const real (&gyn)[5], real rj, real rj1, real vx0, real vx1, real vy0, real vy1, real bj,
                         real bj1, real (&h)[5]) {
            real a4vy = 0, a4by = 0;
            if (cross) {
                const real q = (real)0.25;
                a4vy = ((g.gx[0][m + 1][tm1] + g.gx[0][m + 1][t]) + (g.gx[0][m + 2][tm1] + g.gx[0][m + 2][t])) * q;
                a4by = ((g.gx[1][m + 1][tm1] + g.gx[1][m + 1][t]) + (g.gx[1][m + 2][tm1] + g.gx[1][m + 2][t])) * q;
            }
            const real rf = half * (rj + rj1);
            const real vxf = half * (vx0 + vx1);
            const real vyf = half * (vy0 + vy1);
            const real bxf = half * (bj + bj1);
            const real tyy = rf * gyn[QVY];
            const real tyx = half * rf * (gyn[QVX] + a4vy);
            const real ez = a4by - gyn[QB];
            h[CR] = gyn[QR];
            h[CMX] = tyx;
            h[CMY] = tyy;
            h[CE] = (gyn[QE] + (vyf * tyy + vxf * tyx)) - bxf * ez;
            h[CB] = -ez;
        };
        real hyp[5];
        yflux(j0 - 1, gbot, yat(QR, j0 - 1), u[0].v[0], yat(QVX, j0 - 1), vx[0], yat(QVY, j0 - 1), vy[0],
              yat(QB, j0 - 1), u[0].v[4], hyp);
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int j = j0 + k;
            const bool in = k + 1 < R;
            const int kn = in ? k + 1 : k;
            real hyn[5];
            yflux(j, gy[k], u[k].v[0], in ? u[kn].v[0] : yat(QR, j + 1), vx[k], in ? vx[kn] : yat(QVX, j + 1), vy[k],
                  in ? vy[kn] : yat(QVY, j + 1), u[k].v[4], in ? u[kn].v[4] : yat(QB, j + 1), hyn);
            real hx[5], hl[5];
            {
                real a4vx = 0, a4bx = 0;
                if (cross) {
                    const real q = (real)0.25;
                    const real p0 = k > 0 ? gy[k > 0 ? k - 1 : 0][QVX] : gbot[QVX];
                    const real p1 = k > 0 ? gy[k > 0 ? k - 1 : 0][QB] : gbot[QB];
                    a4vx = ((p0 + gy[k][QVX]) + (g.gy[0][j][tp1] + g.gy[0][j + 1][tp1])) * q;
                    a4bx = ((p1 + gy[k][QB]) + (g.gy[1][j][tp1] + g.gy[1][j + 1][tp1])) * q;
                }
                const real rf = half * ((zero + u[k].v[0]) + (zero + g.q[0][j + 3][tp1]));
                const real vxf = half * (vx[k] + lds.v[0][j + 3][tp1]);
                const real vyf = half * (vy[k] + lds.v[1][j + 3][tp1]);
                const real byf = half * ((zero + u[k].v[5]) + (zero + g.q[3][j + 3][tp1]));
                const real txx = rf * gx[k][QVX];
                const real txy = half * rf * (gx[k][QVY] + a4vx);
                const real ez = gx[k][QB] - a4bx;
                hx[CR] = gx[k][QR];
                hx[CMX] = txx;
                hx[CMY] = txy;
                hx[CE] = (gx[k][QE] + (vxf * txx + vyf * txy)) + byf * ez;
                hx[CB] = ez;
            }
#pragma unroll
            for (int m = 0; m < 5; ++m) hl[m] = lane_left(hx[m]);
            K[k][0] = K[k][0] + ((hx[CR] - hl[CR]) * idx + (hyn[CR] - hyp[CR]) * idy);
            K[k][1] = K[k][1] + ((hx[CMX] - hl[CMX]) * idx + (hyn[CMX] - hyp[CMX]) * idy);
            K[k][2] = K[k][2] + ((hx[CMY] - hl[CMY]) * idx + (hyn[CMY] - hyp[CMY]) * idy);
            K[k][3] = K[k][3] + ((hx[CE] - hl[CE]) * idx + (hyn[CE] - hyp[CE]) * idy);
            K[k][4] = K[k][4] + (zero + (hyn[CB] - hyp[CB]) * idy);
            K[k][5] = K[k][5] + ((hx[CB] - hl[CB]) * idx + zero);
#pragma unroll
            for (int m = 0; m < 5; ++m) hyp[m] = hyn[m];
#pragma unroll
            for (int f = 0; f < 6; ++f) settle(K[k][f]);
        }
    }

    // ================= combine =================
    double cx_t = 0.0, cy_t = 0.0;
    int bad_t = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if (!outrow[k]) continue;
        const int64_t o = oo[k];
        if (STAGE == 1) {
#pragma unroll
            for (int f = 0; f < NF; ++f) a.out1[0][o + f * fs] = u[k].v[f] + hdt * K[k][f];
        } else if (STAGE == 2) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const real uv = pU[k].v[f], s = u[k].v[f];
                a.out1[0][o + f * fs] = uv + hdt * K[k][f];
                a.out2[0][o + f * fs] = (uv + uv) + ((s - uv) + dt * K[k][f]);
            }
        } else if (STAGE == 3) {
#pragma unroll
            for (int f = 0; f < NF; ++f) a.out1[0][o + f * fs] = pU[k].v[f] + dt * K[k][f];
        } else {
            real un[6];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const real av = pU[k].v[f], s = u[k].v[f];
                un[f] = (s + (av - (s + s)) * third) + dt6 * K[k][f];
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
    if (STAGE == 4) {
        raise_speeds(cx_t, cy_t, bad_t, lds.red, a.sc, a.sc->cur ^ 1);
    }
}

}  // namespace sacx
