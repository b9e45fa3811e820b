// sacx3.hip -- the three-dimensional form of the scheme (paper sections 2
// and 8: the code is implemented in 3-D): kernels, host runtime and the
// sacx3_* C ABI.
//
// A stage of RK4 is two launches, which read the cells outside the grid
// (G = 3 on every side) where the boundary has their values:
//
//   k3_faces   the hyper-diffusion face quantities G_d(q) = nu_f(q) d1_f(q) / h_d
//              for the three face directions and the seven quantities of each
//              face set (rho~, eps~, v_x, v_y, v_z and the two field
//              components across the face), on the faces the fluxes need:
//              along d from cell -1 to n_d - 1, across d from -1 to n.  It
//              marches up z over a tile of (x, y) columns: each plane's
//              primitives go to LDS (the x- and y-face coefficient ratios and
//              the compression s take their neighbours there); the z-face
//              ratio takes its six planes from a per-thread register window.
//   k3_stage_hd   L(S) and the RK4 stage combine: ideal fluxes differenced with
//              the fourth-order central difference (x and y fluxes through
//              LDS, the z flux from a register window), the hyper-diffusive
//              face fluxes H_d (hyper-viscous stress, hyper-resistive e.m.f.,
//              the energy they carry) from the stored G and their divergence,
//              then the storage-saving RK4 combine; stage 4 also reduces the
//              wave speeds of the new state.  The G that the x- and y-face
//              fluxes of a plane read are staged in LDS tiles by loads that
//              write LDS directly.
//
// Splitting the stage in two moves the 21 face quantities through HBM: at
// 512^3 336 B per cell for k3_faces and 504-629 B for the stage launch, against
// the 192 B of the stage's own state accesses.  Without hyper-diffusion
// k3_stage is the only launch of a stage; with it the stage launch is
// k3_stage_hd.
//
// Arithmetic: every value is the IEEE operation sequence of the scheme's
// definition in its storage-saving arrangement (divisions by grid constants
// as multiplications by FP64 reciprocals, no contraction: this unit is built
// with -ffp-contract=off), so results are bit-identical to the test oracle's
// low-storage form.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>

#include "sacx3.h"
#include "sacx_internal.h"
#include "sacx_tile.h"

namespace sacx3i {

using sacx::G;
using sacx::SideMap;

constexpr int NF3 = 8;    // evolved fields
constexpr int NQF = 7;    // quantities of one face set
constexpr int kAlign = 256;
constexpr int kPartials = 1024;
constexpr int TXF = 32, TYF = 8;   // column tile of both launches
constexpr int NT = TXF * TYF;

// field slots of the state
enum { FR = 0, FMX = 1, FMY = 2, FMZ = 3, FE = 4, FBX = 5, FBY = 6, FBZ = 7 };
// primitive slots of the face launch's LDS planes
enum { PR = 0, PE = 1, PVX = 2, PVY = 3, PVZ = 4, PBX = 5, PBY = 6, PBZ = 7, NP = 8 };
// G slots of a face set: rho~, eps~, v_x, v_y, v_z, first and second field
// component across the face (x faces: B_y, B_z; y faces: B_x, B_z; z faces:
// B_x, B_y)
enum { GR = 0, GE = 1, GVX = 2, GVY = 3, GVZ = 4, GB1 = 5, GB2 = 6 };

__host__ __device__ constexpr int gclass(int q) { return q == GR ? 0 : (q == GE ? 1 : (q >= GB1 ? 3 : 2)); }

// Storage of one field: nz + 2G planes of ny + 2G rows of `pitch` elements;
// cell (i, j, k), each index from -G, at xoff + i + (j + G) pitch + (k + G) plane.
// xoff puts cell column 0 of every row on a 256-byte boundary.
struct Layout3 {
    int nx, ny, nz;
    int pitch, xoff;
    int64_t plane, field_elems;
    __host__ __device__ int64_t at(int i, int j, int k) const {
        return (int64_t)xoff + i + (int64_t)(j + G) * pitch + (int64_t)(k + G) * plane;
    }
    // byte offset of cell (i, j, k) (every field array is below 4 GiB)
    __device__ uint32_t off(int i, int j, int k) const {
        return (uint32_t)(xoff + i + (j + G) * pitch) * 8u + (uint32_t)(k + G) * (uint32_t)(plane * 8);
    }
};

// step scalars on the device; the wave-speed accumulators hold IEEE bit
// patterns of non-negative doubles (unsigned max is the floating max)
struct Dev3 {
    double t, dt, cmax, t_end, hdt, dt6;
    double kd2[3][4];                 // c2 * h_d * c_max per constant class
    double last_c[3], last_cmax;
    long long steps;
    int cur, active, nonphys, pad;
    sacx::SpeedWord acc[2][sacx::kAcc];   // [slot], the maximum over the words
};

// grid constants, computed once on the host in FP64
struct Consts3 {
    double gamma, gm1, igm1, third;
    double h[3], ih[3], i12[3], i2[3];
    double kds[3][4];                 // cshk * h_d * h_d per constant class
    double cfl, c2[4];
    int act[3];                       // direction has more than one cell
    int pad;
};

struct Face3Args {
    const double *S;   // stage input: field f at S + f * fs
    double *Gf;        // face quantities: (direction d, slot q) at Gf + (7 d + q) * fs
    int64_t fs;
    Layout3 L;
    SideMap mx, my, mz;   // where the cells outside are read
    Consts3 k;
    const Dev3 *sc;
    int tz, ntx, nty;
};

struct Stage3Args {
    const double *S;   // stage input (differenced)
    const double *U;   // step start state (pointwise)
    const double *A;   // RK accumulator (stage 4)
    double *out1;      // stage output
    double *out2;      // accumulator output (stage 2)
    const double *Gf;
    int64_t fs;
    Layout3 L;
    SideMap mx, my, mz;   // where the cells outside are read (as S; U and A are read in the cells only)
    Consts3 k;
    Dev3 *sc;
    int tz, ntx, nty;
    int cross;
};

// The chip hands consecutive blocks to its 8 XCDs in turn.  Blocks are
// renumbered within each strip of planes so that every XCD gets one contiguous
// run of the strip's tiles in row-major order, a patch a few tile rows high:
// the apron that neighbouring tiles share, along x and along y, is then read
// into one L2.  A bijection of the block indices (the remainder of a strip's
// tiles by 8 goes to its first XCDs).
__device__ __forceinline__ int xcd_block(int tiles) {
    const int b = (int)blockIdx.x, strip = b / tiles, i = b - strip * tiles;
    // the XCD is that of the launch's block index; which one a strip starts
    // with does not matter for the runs
    const int x = i % 8, k = i / 8, q = tiles / 8, r = tiles % 8;
    return strip * tiles + (x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k);
}

// Global accesses take a wave-uniform array base plus a 32-bit per-lane byte
// offset (every field array is below 4 GiB), which the compiler turns into
// scalar-base addressing instead of per-lane 64-bit address arithmetic.
__device__ __forceinline__ double ldo(const double *base, uint32_t off) {
    return *(const double *)((const char *)base + off);
}
__device__ __forceinline__ void sto(double *base, uint32_t off, double v) { *(double *)((char *)base + off) = v; }

__device__ __forceinline__ int ring3(int r) { return (r + 3 * 4096) % 3; }

// ---------------------------------------------------------------- face launch

template <int TX, int TY>
struct FaceLds {
    double q[2][NP][TY + 5][TX + 5];   // primitives of planes r, r-1 (by parity) over the tile + apron
    double vz[3][TY + 1][TX + 1];      // v_z over the compression region, ring of 3 planes
    double s[TY + 1][TX + 1];          // compression s of plane r-1
};

template <int TX, int TY>
__global__ __launch_bounds__(TX *TY, 2) void k3_faces(Face3Args a) {
    __shared__ FaceLds<TX, TY> lds;
    constexpr int BX = TX + 5, BY = TY + 5, BOX = BX * BY;
    constexpr int SX = TX + 1, SY = TY + 1, SREG = SX * SY;
    const Dev3 *sc = a.sc;
    if (!sc->active) return;
    const Layout3 L = a.L;
    const Consts3 &kc = a.k;
    const int64_t fs = a.fs;
    const int blk = xcd_block(a.ntx * a.nty);
    const int X0 = -1 + (blk % a.ntx) * TX;
    const int Y0 = -1 + ((blk / a.ntx) % a.nty) * TY;
    const int zb = -1 + (blk / (a.ntx * a.nty)) * a.tz;
    const int ze = min(zb + a.tz, L.nz + 1);
    const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
    const int x = X0 + tx, y = Y0 + ty;
    const bool colv = x <= L.nx && y <= L.ny;
    const bool xf = colv && x <= L.nx - 1;   // owns an x face
    const bool yf = colv && y <= L.ny - 1;   // owns a y face
    const double gm1 = kc.gm1, igm1 = kc.igm1;
    const double half = 0.5, zero = 0.0;
    // the step's coefficients, read once: read where they are used, each
    // would be read again behind the previous face store (which may alias it)
    double kd2[3][4];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int c = 0; c < 4; ++c) kd2[d][c] = sc->kd2[d][c];

    // plane-independent offsets of the thread's points of the box
    constexpr int NPT = (BOX + TX * TY - 1) / (TX * TY);
    uint32_t oxy[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int p = min(tid + i * TX * TY, BOX - 1);
        oxy[i] = L.off(a.mx.at(X0 - 2 + p % BX), a.my.at(Y0 - 2 + p / BX), -G);
    }

    double w[NQF][6];   // z-face set rho~, eps~, v_x, v_y, v_z, B_x, B_y of planes r-5..r
#pragma unroll
    for (int q = 0; q < NQF; ++q)
#pragma unroll
        for (int k = 0; k < 6; ++k) w[q][k] = 0.0;
    double sA = 0.0, sB = 0.0;   // own column's s of planes r-3, r-2

    const int rend = max(min(ze, L.nz) + 2, ze + 1);
    for (int r = zb - 2; r <= rend; ++r) {
        const int slot = r & 1, pslot = slot ^ 1;
        const int rz = a.mz.at(r);
        // ---- P1: plane r over the tile and its apron -> primitives in LDS
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int p = tid + i * TX * TY;
            if (p >= BOX) break;
            const int bx = p % BX, by = p / BX;
            const uint32_t o = oxy[i] + (uint32_t)(rz + G) * (uint32_t)(L.plane * 8);
            const double rt = ldo(a.S, o), mx = ldo(a.S + FMX * fs, o), my = ldo(a.S + FMY * fs, o),
                         mz = ldo(a.S + FMZ * fs, o);
            const double et = ldo(a.S + FE * fs, o), bx_ = ldo(a.S + FBX * fs, o), by_ = ldo(a.S + FBY * fs, o),
                         bz_ = ldo(a.S + FBZ * fs, o);
            const double ir = 1.0 / rt;
            const double ux = mx * ir, uy = my * ir, uz = mz * ir;
            const double kin = half * ((mx * ux + my * uy) + mz * uz);
            const double b2 = (bx_ * bx_ + by_ * by_) + bz_ * bz_;
            const double pk = gm1 * ((et - kin) - half * b2);
            lds.q[slot][PR][by][bx] = rt;
            lds.q[slot][PE][by][bx] = pk * igm1;
            lds.q[slot][PVX][by][bx] = ux;
            lds.q[slot][PVY][by][bx] = uy;
            lds.q[slot][PVZ][by][bx] = uz;
            lds.q[slot][PBX][by][bx] = bx_;
            lds.q[slot][PBY][by][bx] = by_;
            lds.q[slot][PBZ][by][bx] = bz_;
            if (bx >= 2 && bx < 2 + SX && by >= 2 && by < 2 + SY) lds.vz[ring3(r)][by - 2][bx - 2] = uz;
        }
        __syncthreads();
        // ---- P2: own column's z window; compression s of plane r-1
        {
            const int bx = tx + 2, by = ty + 2;
            const int src[NQF] = {PR, PE, PVX, PVY, PVZ, PBX, PBY};
#pragma unroll
            for (int q = 0; q < NQF; ++q) {
#pragma unroll
                for (int k = 0; k < 5; ++k) w[q][k] = w[q][k + 1];
                w[q][5] = lds.q[slot][src[q]][by][bx];
            }
        }
        const bool splane = r - 1 >= zb && r - 1 <= ze;
        if (splane) {
            const int z0 = ring3(r), z2 = ring3(r - 2);
            for (int p = tid; p < SREG; p += TX * TY) {
                const int sx = p % SX, sy = p / SX;
                const int bx = sx + 2, by = sy + 2;
                const double dv = ((lds.q[pslot][PVX][by][bx + 1] - lds.q[pslot][PVX][by][bx - 1]) * kc.i2[0] +
                                   (lds.q[pslot][PVY][by + 1][bx] - lds.q[pslot][PVY][by - 1][bx]) * kc.i2[1]) +
                                  (lds.vz[z0][sy][sx] - lds.vz[z2][sy][sx]) * kc.i2[2];
                lds.s[sy][sx] = fmax(zero, -dv);
            }
        }
        __syncthreads();
        // ---- P3: x and y faces of plane r-1, z face (r-3)+1/2
        const int wpl = r - 1;
        if (wpl >= zb && wpl < ze) {
            if (xf) {
                const int by = ty + 2;
                const double sf = fmax(lds.s[ty][tx], lds.s[ty][tx + 1]);
                const int src[NQF] = {PR, PE, PVX, PVY, PVZ, PBY, PBZ};
                const uint32_t o = L.off(x, y, wpl);
#pragma unroll
                for (int q = 0; q < NQF; ++q) {
                    const double *row = &lds.q[pslot][src[q]][by][0];
                    const double q0 = row[tx], q1 = row[tx + 1], q2 = row[tx + 2], q3 = row[tx + 3],
                                 q4 = row[tx + 4], q5 = row[tx + 5];
                    const double R = sacx::hd_ratio(q0, q1, q2, q3, q4, q5);
                    const int cl = gclass(q);
                    const double nu = kd2[0][cl] * R + kc.kds[0][cl] * sf;
                    sto(a.Gf + (0 * NQF + q) * fs, o, (nu * (q3 - q2)) * kc.ih[0]);
                }
            }
            if (yf) {
                const int bx = tx + 2;
                const double sf = fmax(lds.s[ty][tx], lds.s[ty + 1][tx]);
                const int src[NQF] = {PR, PE, PVX, PVY, PVZ, PBX, PBZ};
                const uint32_t o = L.off(x, y, wpl);
#pragma unroll
                for (int q = 0; q < NQF; ++q) {
                    const double q0 = lds.q[pslot][src[q]][ty][bx], q1 = lds.q[pslot][src[q]][ty + 1][bx],
                                 q2 = lds.q[pslot][src[q]][ty + 2][bx], q3 = lds.q[pslot][src[q]][ty + 3][bx],
                                 q4 = lds.q[pslot][src[q]][ty + 4][bx], q5 = lds.q[pslot][src[q]][ty + 5][bx];
                    const double R = sacx::hd_ratio(q0, q1, q2, q3, q4, q5);
                    const int cl = gclass(q);
                    const double nu = kd2[1][cl] * R + kc.kds[1][cl] * sf;
                    sto(a.Gf + (1 * NQF + q) * fs, o, (nu * (q3 - q2)) * kc.ih[1]);
                }
            }
        }
        const int f = r - 3;
        if (colv && f >= zb && f < ze && f <= L.nz - 1) {
            const double sf = fmax(sA, sB);
            const uint32_t o = L.off(x, y, f);
#pragma unroll
            for (int q = 0; q < NQF; ++q) {
                const double R = sacx::hd_ratio(w[q][0], w[q][1], w[q][2], w[q][3], w[q][4], w[q][5]);
                const int cl = gclass(q);
                const double nu = kd2[2][cl] * R + kc.kds[2][cl] * sf;
                sto(a.Gf + (2 * NQF + q) * fs, o, (nu * (w[q][3] - w[q][2])) * kc.ih[2]);
            }
        }
        if (splane) {
            sA = sB;
            sB = lds.s[ty][tx];
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- stage launch

// pins a value's computation here: without it the compiler moves arithmetic
// down to the value's use and holds all operands until then
__device__ __forceinline__ void settle(double &v) { asm volatile("" : "+v"(v)); }
template <int N>
__device__ __forceinline__ void settle(double (&v)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) settle(v[k]);
}

// state -> primitives, and the parts that every flux of the cell shares
struct Cell3 {
    double rt, mx, my, mz, et, bx, by, bz, ux, uy, uz, pt, bv, ef;
};

__device__ __forceinline__ Cell3 cell3(const double (&s)[NF3], double gm1) {
    const double half = 0.5;
    Cell3 c;
    c.rt = s[FR]; c.mx = s[FMX]; c.my = s[FMY]; c.mz = s[FMZ]; c.et = s[FE];
    c.bx = s[FBX]; c.by = s[FBY]; c.bz = s[FBZ];
    const double ir = 1.0 / c.rt;
    c.ux = c.mx * ir; c.uy = c.my * ir; c.uz = c.mz * ir;
    const double kin = half * ((c.mx * c.ux + c.my * c.uy) + c.mz * c.uz);
    const double b2 = (c.bx * c.bx + c.by * c.by) + c.bz * c.bz;
    const double pk = gm1 * ((c.et - kin) - half * b2);
    c.pt = pk + half * b2;
    c.bv = (c.bx * c.ux + c.by * c.uy) + c.bz * c.uz;
    c.ef = c.et + c.pt;
    return c;
}

// z fluxes of rho, m_x, m_y, m_z, e, B_x, B_y
__device__ __forceinline__ void zflux(const Cell3 &c, double (&f)[7]) {
    f[0] = c.mz;
    f[1] = c.uz * c.mx - c.bz * c.bx;
    f[2] = c.uz * c.my - c.bz * c.by;
    f[3] = (c.uz * c.mz - c.bz * c.bz) + c.pt;
    f[4] = c.uz * c.ef - c.bz * c.bv;
    f[5] = c.uz * c.bx - c.bz * c.ux;
    f[6] = c.uz * c.by - c.bz * c.uy;
}

// the x and y fluxes of a plane's tile and apron
template <int TX, int TY>
struct PlaneLds3 {
    double fx[7][TY + 4][TX + 4];   // x fluxes of rho, m_x, m_y, m_z, e, B_y, B_z
    double fy[7][TY + 4][TX + 4];   // y fluxes of rho, m_x, m_y, m_z, e, B_x, B_z
    double red[4][TX * TY / 64];
};

template <class Lds>
__device__ __forceinline__ void put_fluxes(Lds &lds, int by, int bx, const Cell3 &c) {
    lds.fx[0][by][bx] = c.mx;
    lds.fx[1][by][bx] = (c.ux * c.mx - c.bx * c.bx) + c.pt;
    lds.fx[2][by][bx] = c.ux * c.my - c.bx * c.by;
    lds.fx[3][by][bx] = c.ux * c.mz - c.bx * c.bz;
    lds.fx[4][by][bx] = c.ux * c.ef - c.bx * c.bv;
    lds.fx[5][by][bx] = c.ux * c.by - c.bx * c.uy;
    lds.fx[6][by][bx] = c.ux * c.bz - c.bx * c.uz;
    lds.fy[0][by][bx] = c.my;
    lds.fy[1][by][bx] = c.uy * c.mx - c.by * c.bx;
    lds.fy[2][by][bx] = (c.uy * c.my - c.by * c.by) + c.pt;
    lds.fy[3][by][bx] = c.uy * c.mz - c.by * c.bz;
    lds.fy[4][by][bx] = c.uy * c.ef - c.by * c.bv;
    lds.fy[5][by][bx] = c.uy * c.bx - c.by * c.ux;
    lds.fy[6][by][bx] = c.uy * c.bz - c.by * c.uz;
}

// box position of apron point i (TY + 4 rows of TX + 4 columns without the
// TY x TX tile at (2, 2))
template <int TX, int TY>
__device__ __forceinline__ void frame_point(int i, int &bx, int &by) {
    constexpr int BX = TX + 4;
    if (i < 2 * BX) { by = i / BX; bx = i % BX; }
    else if (i < 4 * BX) { by = TY + 2 + (i - 2 * BX) / BX; bx = (i - 2 * BX) % BX; }
    else { const int j = i - 4 * BX, c4 = j % 4; by = 2 + j / 4; bx = c4 < 2 ? c4 : TX + c4; }
}

// -(D_x F_x + D_y F_y + D_z F_z) of the own cell: x and y fluxes from LDS, the
// z fluxes of planes r-2 .. r+2 (w, fzn)
template <class Lds>
__device__ __forceinline__ void ideal_terms(const Lds &lds, int by, int bx, const Consts3 &kc,
                                            const double (&w)[4][7], const double (&fzn)[7], double (&K)[NF3]) {
    const double eight = 8.0, zero = 0.0;
    double ax[7], ay[7];
    // a batch: the four neighbours of up to four fluxes, read together; left
    // to itself the compiler reads two or four values and waits, for every
    // flux again.
    double q[4][4];
    auto readx = [&](double (&b)[4][4], int k0, int nb) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nb) {
                const double *p = &lds.fx[k0 + k][by][bx];
                b[k][0] = p[-2]; b[k][1] = p[-1]; b[k][2] = p[1]; b[k][3] = p[2];
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto ready = [&](double (&b)[4][4], int k0, int nb) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nb) {
                b[k][0] = lds.fy[k0 + k][by - 2][bx]; b[k][1] = lds.fy[k0 + k][by - 1][bx];
                b[k][2] = lds.fy[k0 + k][by + 1][bx]; b[k][3] = lds.fy[k0 + k][by + 2][bx];
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto diff = [&](const double (&b)[4][4], double *d, int nb, double i12) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nb) {
                d[k] = (eight * (b[k][2] - b[k][1]) - (b[k][3] - b[k][0])) * i12;
                settle(d[k]);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    readx(q, 0, 4);
    diff(q, ax, 4, kc.i12[0]);
    readx(q, 4, 3);
    diff(q, ax + 4, 3, kc.i12[0]);
    ready(q, 0, 4);
    diff(q, ay, 4, kc.i12[1]);
    ready(q, 4, 3);
    diff(q, ay + 4, 3, kc.i12[1]);
    double ab[NF3], ez[NF3];
    ab[FR] = ax[0] + ay[0];
    ab[FMX] = ax[1] + ay[1];
    ab[FMY] = ax[2] + ay[2];
    ab[FMZ] = ax[3] + ay[3];
    ab[FE] = ax[4] + ay[4];
    ab[FBX] = zero + ay[5];
    ab[FBY] = ax[5] + zero;
    ab[FBZ] = ax[6] + ay[6];
#pragma unroll
    for (int f = 0; f < 7; ++f) ez[f] = (eight * (w[3][f] - w[1][f]) - (fzn[f] - w[0][f])) * kc.i12[2];
    ez[FBZ] = zero;
#pragma unroll
    for (int f = 0; f < NF3; ++f) K[f] = -(ab[f] + ez[f]);
}

// wave speeds and physicality of the states a thread wrote at stage 4
struct Speeds3 {
    double c[3] = {0.0, 0.0, 0.0};
    int bad = 0;
    __device__ __forceinline__ void add(const double (&un)[NF3], double gm1, double gamma) {
        const double half = 0.5;
        const double ir = 1.0 / un[FR];
        const double ux = un[FMX] * ir, uy = un[FMY] * ir, uz = un[FMZ] * ir;
        const double kin = half * ((un[FMX] * ux + un[FMY] * uy) + un[FMZ] * uz);
        const double b2 = (un[FBX] * un[FBX] + un[FBY] * un[FBY]) + un[FBZ] * un[FBZ];
        const double pk = gm1 * ((un[FE] - kin) - half * b2);
        const double cf = sqrt((gamma * pk + b2) * ir);
        bool fin = isfinite(cf);
#pragma unroll
        for (int f = 0; f < NF3; ++f) fin = fin && isfinite(un[f]);
        if (!(un[FR] > 0.0) || !(pk > 0.0) || !fin) {
            bad = 1;
        } else {
            c[0] = fmax(c[0], fabs(ux) + cf);
            c[1] = fmax(c[1], fabs(uy) + cf);
            c[2] = fmax(c[2], fabs(uz) + cf);
        }
    }
    // one result per wave into red (wave wv)
    template <int NW>
    __device__ __forceinline__ void reduce(double (&red)[4][NW], int wv, int lane) {
#pragma unroll
        for (int d = 0; d < 3; ++d) c[d] = sacx::wave_max(c[d]);
        const bool any = __any(bad) != 0;
        if (lane == 63) {
#pragma unroll
            for (int d = 0; d < 3; ++d) red[d][wv] = c[d];
            red[3][wv] = any ? 1.0 : 0.0;
        }
    }
};

template <int NW>
__device__ __forceinline__ void raise_speeds(const double (&red)[4][NW], Dev3 *sc, int slot) {
    if (threadIdx.x >= 4) return;
    double m = 0.0;
    for (int k = 0; k < NW; ++k) m = fmax(m, red[threadIdx.x][k]);
    if (threadIdx.x < 3)
        atomicMax(&sc->acc[slot][sacx::acc_word()].v[threadIdx.x], (unsigned long long)__double_as_longlong(m));
    else if (m > 0.0)
        atomicOr(&sc->nonphys, 1);
}

// the RK4 combine of the own cell at byte offset o: so is the stage input,
// uo U (stages 2, 3) or A (stage 4); un is the state written at stage 4
template <int STAGE>
__device__ __forceinline__ void combine3(const Stage3Args &a, int64_t fs, uint32_t o, const double (&so)[NF3],
                                         const double (&uo)[NF3], const double (&K)[NF3], double dt, double hdt,
                                         double dt6, double (&un)[NF3]) {
#pragma unroll
    for (int f = 0; f < NF3; ++f) {
        if (STAGE == 1) {
            sto(a.out1 + f * fs, o, so[f] + hdt * K[f]);
        } else if (STAGE == 2) {
            const double u = uo[f], sv = so[f];
            sto(a.out1 + f * fs, o, u + hdt * K[f]);
            sto(a.out2 + f * fs, o, (u + u) + ((sv - u) + dt * K[f]));
        } else if (STAGE == 3) {
            sto(a.out1 + f * fs, o, uo[f] + dt * K[f]);
        } else {
            const double av = uo[f], sv = so[f];
            un[f] = (sv + (av - (sv + sv)) * a.k.third) + dt6 * K[f];
            sto(a.out1 + f * fs, o, un[f]);
        }
    }
}

// without hyper-diffusion: one thread per column of the tile.  Starting the z
// fluxes from four planes read before the loop instead of four warm-up planes
// took 256^3 from 4.85 to 4.03 ms per step, 100 x 90 x 80 from 0.322 to 0.300.
template <int STAGE, int TX, int TY>
__global__ __launch_bounds__(TX *TY, 1) void k3_stage(Stage3Args a) {
    __shared__ PlaneLds3<TX, TY> lds;
    constexpr int BX = TX + 4, BY = TY + 4;
    constexpr int NFRAME = BX * BY - TX * TY;
    Dev3 *sc = a.sc;
    if (!sc->active) return;
    const Layout3 L = a.L;
    const Consts3 &kc = a.k;
    const int64_t fs = a.fs;
    const int blk = xcd_block(a.ntx * a.nty);
    const int X0 = (blk % a.ntx) * TX;
    const int Y0 = ((blk / a.ntx) % a.nty) * TY;
    const int zb = (blk / (a.ntx * a.nty)) * a.tz;
    const int ze = min(zb + a.tz, L.nz);
    const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
    const int x = X0 + tx, y = Y0 + ty;
    const bool colv = x < L.nx && y < L.ny;
    const double dt = sc->dt, hdt = sc->hdt, dt6 = sc->dt6;
    const double *usrc = STAGE == 4 ? a.A : a.U;
    // the streamed column: the thread's own (x, y), mapped like every box point
    const int cx = a.mx.at(x), cy = a.my.at(y);
    auto column = [&](int k, double (&s)[NF3]) __attribute__((always_inline)) {
        const uint32_t o = L.off(cx, cy, a.mz.at(k));
#pragma unroll
        for (int f = 0; f < NF3; ++f) s[f] = ldo(a.S + f * fs, o);
    };
    double fzw[4][7];   // z fluxes of planes r-2..r+1
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        double s[NF3];
        column(zb - 2 + m, s);
        zflux(cell3(s, kc.gm1), fzw[m]);
    }
    Speeds3 sp;
    // state of the own column, plane r+2, loaded one plane early
    double psn[NF3];
    column(zb + 2, psn);

    for (int r = zb; r < ze; ++r) {
        double so[NF3];   // own cell's stage input (the combine's pointwise operand)
        for (int p = tid; p < TX * TY + NFRAME; p += TX * TY) {
            int bx = tx + 2, by = ty + 2;
            if (p >= TX * TY) frame_point<TX, TY>(p - TX * TY, bx, by);
            const uint32_t o = L.off(a.mx.at(X0 - 2 + bx), a.my.at(Y0 - 2 + by), r);
            double s[NF3];
#pragma unroll
            for (int f = 0; f < NF3; ++f) s[f] = ldo(a.S + f * fs, o);
            if (p < TX * TY) {
#pragma unroll
                for (int f = 0; f < NF3; ++f) so[f] = s[f];
            }
            put_fluxes(lds, by, bx, cell3(s, kc.gm1));
        }
        __syncthreads();
        double fzn[7];
        zflux(cell3(psn, kc.gm1), fzn);
        column(r + 3, psn);   // past the block's last plane: ghost planes, unused
        __builtin_amdgcn_sched_barrier(0);
        if (colv) {
            double K[NF3], uo[NF3], un[NF3];
            ideal_terms(lds, ty + 2, tx + 2, kc, fzw, fzn, K);
            const uint32_t oo = L.off(x, y, r);
            if (STAGE > 1) {
#pragma unroll
                for (int f = 0; f < NF3; ++f) uo[f] = ldo(usrc + f * fs, oo);
            }
            combine3<STAGE>(a, fs, oo, so, uo, K, dt, hdt, dt6, un);
            if (STAGE == 4) sp.add(un, kc.gm1, kc.gamma);
        }
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            fzw[0][k] = fzw[1][k]; fzw[1][k] = fzw[2][k]; fzw[2][k] = fzw[3][k]; fzw[3][k] = fzn[k];
        }
        __syncthreads();
    }

    if (STAGE == 4) {
        sp.reduce(lds.red, tid >> 6, tid & 63);
        __syncthreads();
        raise_speeds(lds.red, sc, sc->cur ^ 1);
    }
}

template <int TX, int TY>
struct StageLds3 {
    double pr[7][TY + 4][TX + 4];   // rho, v_x, v_y, v_z, B_x, B_y, B_z of plane r
    double fx[7][TY + 4][TX + 4];   // as in PlaneLds3
    double fy[7][TY + 4][TX + 4];
    // the face quantities the face fluxes of plane r read, staged from the
    // face arrays once per plane: element [.][j][i] is the face stored at
    // (X0 - 2 + i, Y0 - 1 + j).  Rows are GW = TX + 4 doubles, filled as
    // 16-byte pairs from an even x, 128 doubles per wave instruction; each
    // tile is padded to whole instructions.
    static constexpr int GW = TX + 4;
    static constexpr int fill128(int rows) { return (rows * GW + 127) / 128 * 128; }
    struct GzTile {
        alignas(16) double v[4][TY + 2][GW];   // G_z of v_x, B_x, v_y, B_y
        double pad[fill128(4 * (TY + 2)) - 4 * (TY + 2) * GW + 2];
    };
    alignas(16) double gx[NQF][TY + 2][GW];    // G_x, all seven, plane r
    double gx_pad[fill128(NQF * (TY + 2)) - NQF * (TY + 2) * GW + 2];
    alignas(16) double gy[NQF][TY + 1][GW];    // G_y, all seven, plane r
    double gy_pad[fill128(NQF * (TY + 1)) - NQF * (TY + 1) * GW + 2];
    GzTile gz[2];                              // planes r-1 and r (by parity)
    // between the roles, one slot per column: rho, v, B of plane r+1 for the
    // H role's z face, then the hyper-diffusive terms of plane r for the P
    // role.  A slot is used by one thread of each role, in turn.
    double ex[NF3][TX * TY];
    double red[4][TX * TY / 64];
};

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;

// Fill an LDS tile of face quantities with loads that write LDS directly: no
// registers hold the data, and the loads overlap whatever the wave does until
// it waits for them.  The tile holds NQ quantities x H rows
// x GW columns; row j of quantity q is slot q of direction d (for the G_z
// tile, its q-th of v_x, B_x, v_y, B_y) at y = Y0 - 1 + j, x = X0 - 2 ..
// X0 - 3 + GW, plane k.  Lane l of a wave instruction moves the pair p =
// 64 c + l of the tile (two doubles, 16-byte aligned in both memories: x is
// even and column 0 of every row is on a 256-byte boundary); lanes past the
// tile repeat its last pair into the padding.  Positions past the ghost
// layers read whatever follows in the array (a later row or plane: staged
// planes end at n_z - 1 and three ghost planes follow); no output reads them.
// Wave wv of NWAVE takes the instructions wv, wv + NWAVE, ...; their sources
// are formed once (for the first plane) and moved up plane by plane.
template <int NQ, int H, int GW, bool ZSEL, int NWAVE>
struct dma_tile {
    static constexpr int PR = GW / 2, NP = NQ * H * PR, NCH = (NP + 63) / 64, NI = (NCH + NWAVE - 1) / NWAVE;
    static_assert(GW % 2 == 0, "rows are filled in pairs");
    const char *src[NI];
    __device__ __forceinline__ dma_tile(const double *Gf, int64_t fs, const Layout3 &L, int d, int X0, int Y0, int k,
                                        int wv, int lane) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int p = min((wv + i * NWAVE) * 64 + lane, NP - 1);
            const int row = p / PR, pr = p - row * PR;
            const int q = row / H, j = row - q * H;
            const int qs = ZSEL ? (q == 0 ? GVX : (q == 1 ? GB1 : (q == 2 ? GVY : GB2))) : q;
            src[i] = (const char *)(Gf + (int64_t)(NQF * d + qs) * fs) + L.off(X0 - 2 + 2 * pr, Y0 - 1 + j, k);
        }
    }
    // fill dst from the current plane and move to the next
    __device__ __forceinline__ void fill(double *dst, int wv, uint32_t plane_bytes) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int c = wv + i * NWAVE;
            if (c < NCH) __builtin_amdgcn_global_load_lds((glb_void *)src[i], (lds_void *)(dst + c * 128), 16, 0, 0);
            src[i] += plane_bytes;
        }
    }
};

// the eight face fluxes of one face from its seven G values, the cross-term
// means A4 of the two other directions (first, second in x, y, z order) and
// the face means of rho, v and B; d is the face direction
struct FaceFlux {
    double h[NF3];
};

template <int D>
__device__ __forceinline__ FaceFlux face_flux(const double (&g)[NQF], double a4v1, double a4b1, double a4v2,
                                              double a4b2, double rf, const double (&vf)[3], const double (&bf)[3]) {
    // the two directions other than D, in x, y, z order
    constexpr int O1 = D == 0 ? 1 : 0, O2 = D == 2 ? 1 : 2;
    const double half = 0.5;
    double tau[3], hb[3];
    tau[D] = rf * g[GVX + D];
    hb[D] = 0.0;
    tau[O1] = half * rf * (g[GVX + O1] + a4v1);
    tau[O2] = half * rf * (g[GVX + O2] + a4v2);
    hb[O1] = g[GB1] - a4b1;
    hb[O2] = g[GB2] - a4b2;
    const double work = (vf[D] * tau[D] + vf[O1] * tau[O1]) + vf[O2] * tau[O2];
    const double mag = bf[O1] * hb[O1] + bf[O2] * hb[O2];
    FaceFlux H;
    H.h[FR] = g[GR];
    H.h[FMX] = tau[0];
    H.h[FMY] = tau[1];
    H.h[FMZ] = tau[2];
    H.h[FE] = (g[GE] + work) + mag;
    H.h[FBX] = hb[0];
    H.h[FBY] = hb[1];
    H.h[FBZ] = hb[2];
    return H;
}

// LDS between the roles: the wave's own LDS accesses are complete before it
// arrives, loads from memory stay in flight (the fills of the face tiles are
// waited for where they are needed, by the waves that issued them)
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// With hyper-diffusion a tile's columns have two threads each, in different
// waves: the P role (waves 0 .. NW-1) keeps the column's states and z fluxes,
// takes the ideal terms and the combine; the H role fills the face tiles,
// takes the apron of the plane and all face fluxes of the cell.
//
// Bound by latency and memory: per cell it reads the 8 fields, the 21 face
// quantities and at stages 2-4 the 8 stored operands, and writes 8 or 16
// values.  With one thread per column it took 256 VGPRs, 148-190 AGPRs and so
// one wave per SIMD, whose waves waited in 42 % of their cycles; each plane's
// state was also read twice (for the plane's x and y terms, and two planes
// early for the z fluxes).  Two roles with a loop each fit two waves per SIMD
// (219-241 VGPRs, 153 KB of LDS), and the P role has the registers to keep a
// state until its plane comes.  256^3 FP64, per launch: 2.65-3.0 -> 1.67-2.0 ms;
// two whole steps 35.78 -> 27.68 ms; five of 75 x 53 x 61: 2.52 -> 2.03 ms.
// The order of the LDS reads is fixed in the source: read two at a time, each
// pair waited for, a launch took 1.79-2.19 ms; in batches 1.62-2.03 ms; a whole
// face's 37 values in one batch spilled (2.4-2.7 ms).
template <int STAGE, int TX, int TY>
__global__ __launch_bounds__(2 * TX *TY, 1) void k3_stage_hd(Stage3Args a) {
    __shared__ StageLds3<TX, TY> lds;
    constexpr int BX = TX + 4, BY = TY + 4, NCOL = TX * TY, NW = NCOL / 64;
    constexpr int NFRAME = BX * BY - NCOL;
    static_assert(NFRAME <= NCOL, "one apron point per thread of the H role");
    Dev3 *sc = a.sc;
    if (!sc->active) return;
    const Layout3 L = a.L;
    const Consts3 &kc = a.k;
    const int64_t fs = a.fs;
    const int blk = xcd_block(a.ntx * a.nty);
    const int X0 = (blk % a.ntx) * TX;
    const int Y0 = ((blk / a.ntx) % a.nty) * TY;
    const int zb = (blk / (a.ntx * a.nty)) * a.tz;
    const int ze = min(zb + a.tz, L.nz);
    const int wvb = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const bool prole = wvb < NW;
    const int wv = prole ? wvb : wvb - NW;
    const int tid = wv * 64 + lane, tx = tid % TX, ty = tid / TX;
    const int x = X0 + tx, y = Y0 + ty, bx = tx + 2, by = ty + 2;
    const double half = 0.5;

    if (prole) {
        const bool colv = x < L.nx && y < L.ny;
        const int xc = min(x, L.nx - 1), yc = min(y, L.ny - 1);   // column clamped into the cells
        // the streamed column: the thread's own (x, y), mapped like every
        // box point, so that columns past the last cell hold the values
        // their neighbours difference
        const int cx = a.mx.at(x), cy = a.my.at(y);
        const double dt = sc->dt, hdt = sc->hdt, dt6 = sc->dt6;
        const double *usrc = STAGE == 4 ? a.A : a.U;
        auto column = [&](int k, double (&s)[NF3]) __attribute__((always_inline)) {
            const uint32_t o = L.off(cx, cy, a.mz.at(k));
#pragma unroll
            for (int f = 0; f < NF3; ++f) s[f] = ldo(a.S + f * fs, o);
        };
        auto operand = [&](int k, double (&u)[NF3]) __attribute__((always_inline)) {
            const uint32_t o = L.off(xc, yc, k);
#pragma unroll
            for (int f = 0; f < NF3; ++f) u[f] = ldo(usrc + f * fs, o);
        };
        auto hand = [&](const Cell3 &c) __attribute__((always_inline)) {
            lds.ex[0][tid] = c.rt;
            lds.ex[1][tid] = c.ux; lds.ex[2][tid] = c.uy; lds.ex[3][tid] = c.uz;
            lds.ex[4][tid] = c.bx; lds.ex[5][tid] = c.by; lds.ex[6][tid] = c.bz;
        };
        double fzw[4][7];                  // z fluxes of planes r-2..r+1
        double s0[NF3], s1[NF3], s2[NF3];  // the column's states of planes r, r+1, r+2
        double uo[NF3];                    // the combine's stored operand of plane r
        column(zb - 2, s0);
        column(zb - 1, s1);
        zflux(cell3(s0, kc.gm1), fzw[0]);
        zflux(cell3(s1, kc.gm1), fzw[1]);
        column(zb, s0);
        column(zb + 1, s1);
        column(zb + 2, s2);
        zflux(cell3(s0, kc.gm1), fzw[2]);
        const Cell3 c1 = cell3(s1, kc.gm1);
        zflux(c1, fzw[3]);
        hand(c1);
        if (STAGE > 1) operand(zb, uo);
        Speeds3 sp;
        for (int r = zb; r < ze; ++r) {
            const Cell3 c = cell3(s0, kc.gm1);
            lds.pr[0][by][bx] = c.rt;
            lds.pr[1][by][bx] = c.ux; lds.pr[2][by][bx] = c.uy; lds.pr[3][by][bx] = c.uz;
            lds.pr[4][by][bx] = c.bx; lds.pr[5][by][bx] = c.by; lds.pr[6][by][bx] = c.bz;
            put_fluxes(lds, by, bx, c);
            lds_barrier();
            // state of plane r+3 (past the block's last plane: ghost planes,
            // unused), consumed one plane later
            double s3[NF3], fzn[7], K[NF3], un[NF3];
            column(r + 3, s3);
            const Cell3 c2 = cell3(s2, kc.gm1);
            zflux(c2, fzn);
            settle(fzn);
            ideal_terms(lds, by, bx, kc, fzw, fzn, K);
            settle(K);
            lds_barrier();
#pragma unroll
            for (int f = 0; f < NF3; ++f) K[f] = K[f] + lds.ex[f][tid];
            hand(c2);
            if (colv) {
                combine3<STAGE>(a, fs, L.off(x, y, r), s0, uo, K, dt, hdt, dt6, un);
                if (STAGE == 4) sp.add(un, kc.gm1, kc.gamma);
            }
            if (STAGE > 1) operand(r + 1, uo);
#pragma unroll
            for (int f = 0; f < NF3; ++f) { s0[f] = s1[f]; s1[f] = s2[f]; s2[f] = s3[f]; }
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                fzw[0][k] = fzw[1][k]; fzw[1][k] = fzw[2][k]; fzw[2][k] = fzw[3][k]; fzw[3][k] = fzn[k];
            }
        }
        if (STAGE == 4) sp.reduce(lds.red, wv, lane);
    } else {
        const bool cross = a.cross != 0;
        const double *Gf = a.Gf;
        auto garr = [&](int d, int q) { return Gf + (int64_t)(NQF * d + q) * fs; };
        const uint32_t sy = (uint32_t)L.pitch * 8u, sz = (uint32_t)(L.plane * 8);   // byte strides
        // columns past the last cell read a cell of the block and discard it
        const int xc = min(x, L.nx - 1), yc = min(y, L.ny - 1);
        dma_tile<NQF, TY + 2, TX + 4, false, NW> tgx(Gf, fs, L, 0, X0, Y0, zb, wv, lane);
        dma_tile<NQF, TY + 1, TX + 4, false, NW> tgy(Gf, fs, L, 1, X0, Y0, zb, wv, lane);
        dma_tile<4, TY + 2, TX + 4, true, NW> tgz(Gf, fs, L, 2, X0, Y0, zb - 1, wv, lane);
        tgz.fill(&lds.gz[(zb - 1) & 1].v[0][0][0], wv, sz);
        // apron point of this thread
        const bool fr = tid < NFRAME;
        int fbx = 0, fby = 0;
        frame_point<TX, TY>(fr ? tid : 0, fbx, fby);
        const int fgx = a.mx.at(X0 - 2 + fbx), fgy = a.my.at(Y0 - 2 + fby);
        double sf[NF3];   // its state of the next plane
        auto apron = [&](int k) __attribute__((always_inline)) {
            const uint32_t o = L.off(fgx, fgy, a.mz.at(k));
#pragma unroll
            for (int f = 0; f < NF3; ++f) sf[f] = ldo(a.S + f * fs, o);
        };
        if (fr) apron(zb);
        // what the z face r+1/2 reads beyond the tiles of plane r: G_z of
        // rho~, eps~ and v_z, and G_x, G_y of v_z and B_z of plane r+1 around
        // it (x faces x-1, x, then y faces y-1, y); loaded one plane early
        double pgz[3], pgc[4][2];
        auto zface = [&](int k) __attribute__((always_inline)) {
            const uint32_t c = L.off(xc, yc, k);
            pgz[0] = ldo(garr(2, GR), c);
            pgz[1] = ldo(garr(2, GE), c);
            pgz[2] = ldo(garr(2, GVZ), c);
            if (cross) {
                pgc[0][0] = ldo(garr(0, GVZ), c - 8u + sz); pgc[0][1] = ldo(garr(0, GVZ), c + sz);
                pgc[1][0] = ldo(garr(0, GB2), c - 8u + sz); pgc[1][1] = ldo(garr(0, GB2), c + sz);
                pgc[2][0] = ldo(garr(1, GVZ), c - sy + sz); pgc[2][1] = ldo(garr(1, GVZ), c + sz);
                pgc[3][0] = ldo(garr(1, GB2), c - sy + sz); pgc[3][1] = ldo(garr(1, GB2), c + sz);
            }
        };
        // H_z of face zb-1/2, everything from memory
        FaceFlux hzp;
        {
            const uint32_t c = L.off(xc, yc, zb - 1), cs = L.off(xc, yc, a.mz.at(zb - 1));
            double sa[NF3], sb[NF3], g[NQF];
#pragma unroll
            for (int f = 0; f < NF3; ++f) { sa[f] = ldo(a.S + f * fs, cs); sb[f] = ldo(a.S + f * fs, c + sz); }
#pragma unroll
            for (int q = 0; q < NQF; ++q) g[q] = ldo(garr(2, q), c);
            double v1 = 0.0, b1 = 0.0, v2 = 0.0, b2 = 0.0;
            if (cross) {
                auto mean = [&](const double *A, uint32_t st) __attribute__((always_inline)) {
                    return ((ldo(A, c - st) + ldo(A, c)) + (ldo(A, c - st + sz) + ldo(A, c + sz))) * 0.25;
                };
                v1 = mean(garr(0, GVZ), 8u);
                b1 = mean(garr(0, GB2), 8u);
                v2 = mean(garr(1, GVZ), sy);
                b2 = mean(garr(1, GB2), sy);
            }
            const Cell3 ca = cell3(sa, kc.gm1), cb = cell3(sb, kc.gm1);
            const double rf = half * (ca.rt + cb.rt);
            const double vf[3] = {half * (ca.ux + cb.ux), half * (ca.uy + cb.uy), half * (ca.uz + cb.uz)};
            const double bf[3] = {half * (ca.bx + cb.bx), half * (ca.by + cb.by), half * (ca.bz + cb.bz)};
            hzp = face_flux<2>(g, v1, b1, v2, b2, rf, vf, bf);
        }
        zface(zb);
        for (int r = zb; r < ze; ++r) {
            const int zc = r & 1, zp = zc ^ 1;   // G_z slots of planes r and r-1
            tgx.fill(&lds.gx[0][0][0], wv, sz);
            tgy.fill(&lds.gy[0][0][0], wv, sz);
            tgz.fill(&lds.gz[zc].v[0][0][0], wv, sz);
            if (fr) {
                const Cell3 c = cell3(sf, kc.gm1);
                lds.pr[0][fby][fbx] = c.rt;
                lds.pr[1][fby][fbx] = c.ux; lds.pr[2][fby][fbx] = c.uy; lds.pr[3][fby][fbx] = c.uz;
                lds.pr[4][fby][fbx] = c.bx; lds.pr[5][fby][fbx] = c.by; lds.pr[6][fby][fbx] = c.bz;
                put_fluxes(lds, fby, fbx, c);
            }
            loads_done();   // the tiles
            lds_barrier();
            double T[NF3];
            {   // H_z on the face r+1/2
                const int j = ty + 1, i = tx + 2;
                double g[NQF];
                g[GR] = pgz[0]; g[GE] = pgz[1]; g[GVZ] = pgz[2];
                g[GVX] = lds.gz[zc].v[0][j][i];
                g[GB1] = lds.gz[zc].v[1][j][i];
                g[GVY] = lds.gz[zc].v[2][j][i];
                g[GB2] = lds.gz[zc].v[3][j][i];
                double v1 = 0.0, b1 = 0.0, v2 = 0.0, b2 = 0.0;
                if (cross) {
                    // means of the four x faces (G of v_z, B_z), then y faces
                    v1 = ((lds.gx[GVZ][j][i - 1] + lds.gx[GVZ][j][i]) + (pgc[0][0] + pgc[0][1])) * 0.25;
                    b1 = ((lds.gx[GB2][j][i - 1] + lds.gx[GB2][j][i]) + (pgc[1][0] + pgc[1][1])) * 0.25;
                    v2 = ((lds.gy[GVZ][j - 1][i] + lds.gy[GVZ][j][i]) + (pgc[2][0] + pgc[2][1])) * 0.25;
                    b2 = ((lds.gy[GB2][j - 1][i] + lds.gy[GB2][j][i]) + (pgc[3][0] + pgc[3][1])) * 0.25;
                }
                const double rf = half * (lds.pr[0][by][bx] + lds.ex[0][tid]);
                double vf[3], bf[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    vf[k] = half * (lds.pr[1 + k][by][bx] + lds.ex[1 + k][tid]);
                    bf[k] = half * (lds.pr[4 + k][by][bx] + lds.ex[4 + k][tid]);
                }
                const FaceFlux hz = face_flux<2>(g, v1, b1, v2, b2, rf, vf, bf);
#pragma unroll
                for (int f = 0; f < NF3; ++f) T[f] = (hz.h[f] - hzp.h[f]) * kc.ih[2];
                hzp = hz;
            }
            settle(T);
            settle(hzp.h);
            __builtin_amdgcn_sched_barrier(0);
            zface(r + 1);
            if (fr) apron(r + 1);
            __builtin_amdgcn_sched_barrier(0);
            // H_x on the faces x-1/2 and x+1/2, then H_y on y-1/2 and y+1/2,
            // one face at a time (a scheduling barrier after each keeps the
            // LDS reads of later faces out of the registers of earlier ones),
            // in two batches of reads, the cross terms' and the rest
            double ah[NF3], bh[NF3];
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int lb = bx - 1 + side;         // box column of the face's left cell xx = x - 1 + side
                const int i = tx + side + 1;          // staged column of xx
                double v1 = 0.0, b1 = 0.0, v2 = 0.0, b2 = 0.0;
                if (cross) {
                    double n[4][4];
                    // y faces around the x face (G of v_x, B_x): (xx, y-1), (xx, y),
                    // (xx+1, y-1), (xx+1, y); then z faces: (xx, r-1), (xx, r),
                    // (xx+1, r-1), (xx+1, r)
                    n[0][0] = lds.gy[GVX][ty][i]; n[0][1] = lds.gy[GVX][ty + 1][i];
                    n[0][2] = lds.gy[GVX][ty][i + 1]; n[0][3] = lds.gy[GVX][ty + 1][i + 1];
                    n[1][0] = lds.gy[GB1][ty][i]; n[1][1] = lds.gy[GB1][ty + 1][i];
                    n[1][2] = lds.gy[GB1][ty][i + 1]; n[1][3] = lds.gy[GB1][ty + 1][i + 1];
                    n[2][0] = lds.gz[zp].v[0][ty + 1][i]; n[2][1] = lds.gz[zc].v[0][ty + 1][i];
                    n[2][2] = lds.gz[zp].v[0][ty + 1][i + 1]; n[2][3] = lds.gz[zc].v[0][ty + 1][i + 1];
                    n[3][0] = lds.gz[zp].v[1][ty + 1][i]; n[3][1] = lds.gz[zc].v[1][ty + 1][i];
                    n[3][2] = lds.gz[zp].v[1][ty + 1][i + 1]; n[3][3] = lds.gz[zc].v[1][ty + 1][i + 1];
                    __builtin_amdgcn_sched_barrier(0);
                    v1 = ((n[0][0] + n[0][1]) + (n[0][2] + n[0][3])) * 0.25;
                    b1 = ((n[1][0] + n[1][1]) + (n[1][2] + n[1][3])) * 0.25;
                    v2 = ((n[2][0] + n[2][1]) + (n[2][2] + n[2][3])) * 0.25;
                    b2 = ((n[3][0] + n[3][1]) + (n[3][2] + n[3][3])) * 0.25;
                    settle(v1); settle(b1); settle(v2); settle(b2);
                }
                double g[NQF];
#pragma unroll
                for (int q = 0; q < NQF; ++q) g[q] = lds.gx[q][ty + 1][i];
                double pl[7], ph[7];
#pragma unroll
                for (int k = 0; k < 7; ++k) { pl[k] = lds.pr[k][by][lb]; ph[k] = lds.pr[k][by][lb + 1]; }
                __builtin_amdgcn_sched_barrier(0);
                const double rf = half * (pl[0] + ph[0]);
                double vf[3], bf[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    vf[k] = half * (pl[1 + k] + ph[1 + k]);
                    bf[k] = half * (pl[4 + k] + ph[4 + k]);
                }
                const FaceFlux h = face_flux<0>(g, v1, b1, v2, b2, rf, vf, bf);
#pragma unroll
                for (int f = 0; f < NF3; ++f) ah[f] = side == 0 ? h.h[f] : (h.h[f] - ah[f]) * kc.ih[0];
                settle(ah);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int lb = by - 1 + side;         // box row of the face's lower cell yy = y - 1 + side
                const int j = ty + side;              // staged row of yy
                double v1 = 0.0, b1 = 0.0, v2 = 0.0, b2 = 0.0;
                if (cross) {
                    double n[4][4];
                    // x faces around the y face (G of v_y, B_y): (x-1, yy), (x, yy),
                    // (x-1, yy+1), (x, yy+1); then z faces: (yy, r-1), (yy, r),
                    // (yy+1, r-1), (yy+1, r)
                    n[0][0] = lds.gx[GVY][j][tx + 1]; n[0][1] = lds.gx[GVY][j][tx + 2];
                    n[0][2] = lds.gx[GVY][j + 1][tx + 1]; n[0][3] = lds.gx[GVY][j + 1][tx + 2];
                    n[1][0] = lds.gx[GB1][j][tx + 1]; n[1][1] = lds.gx[GB1][j][tx + 2];
                    n[1][2] = lds.gx[GB1][j + 1][tx + 1]; n[1][3] = lds.gx[GB1][j + 1][tx + 2];
                    n[2][0] = lds.gz[zp].v[2][j][tx + 2]; n[2][1] = lds.gz[zc].v[2][j][tx + 2];
                    n[2][2] = lds.gz[zp].v[2][j + 1][tx + 2]; n[2][3] = lds.gz[zc].v[2][j + 1][tx + 2];
                    n[3][0] = lds.gz[zp].v[3][j][tx + 2]; n[3][1] = lds.gz[zc].v[3][j][tx + 2];
                    n[3][2] = lds.gz[zp].v[3][j + 1][tx + 2]; n[3][3] = lds.gz[zc].v[3][j + 1][tx + 2];
                    __builtin_amdgcn_sched_barrier(0);
                    v1 = ((n[0][0] + n[0][1]) + (n[0][2] + n[0][3])) * 0.25;
                    b1 = ((n[1][0] + n[1][1]) + (n[1][2] + n[1][3])) * 0.25;
                    v2 = ((n[2][0] + n[2][1]) + (n[2][2] + n[2][3])) * 0.25;
                    b2 = ((n[3][0] + n[3][1]) + (n[3][2] + n[3][3])) * 0.25;
                    settle(v1); settle(b1); settle(v2); settle(b2);
                }
                double g[NQF];
#pragma unroll
                for (int q = 0; q < NQF; ++q) g[q] = lds.gy[q][j][tx + 2];
                double pl[7], ph[7];
#pragma unroll
                for (int k = 0; k < 7; ++k) { pl[k] = lds.pr[k][lb][bx]; ph[k] = lds.pr[k][lb + 1][bx]; }
                __builtin_amdgcn_sched_barrier(0);
                const double rf = half * (pl[0] + ph[0]);
                double vf[3], bf[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    vf[k] = half * (pl[1 + k] + ph[1 + k]);
                    bf[k] = half * (pl[4 + k] + ph[4 + k]);
                }
                const FaceFlux h = face_flux<1>(g, v1, b1, v2, b2, rf, vf, bf);
#pragma unroll
                for (int f = 0; f < NF3; ++f) bh[f] = side == 0 ? h.h[f] : (h.h[f] - bh[f]) * kc.ih[1];
                settle(bh);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int f = 0; f < NF3; ++f) lds.ex[f][tid] = (ah[f] + bh[f]) + T[f];
            lds_barrier();
        }
    }

    if (STAGE == 4) {
        lds_barrier();
        raise_speeds(lds.red, sc, sc->cur ^ 1);
    }
}

// ---------------------------------------------------------------- small kernels

// ghost fills (for periodic directions of 1 or 2 cells): x over the cell rows and planes, then y over the padded x
// width, then z over the padded x and y extents (edges and corners filled);
// periodic images or zero-gradient copies
__global__ void k3_fill_x(double *S, int64_t fs, Layout3 L, int pm, int pp, const Dev3 *sc) {
    if (!sc->active) return;
    const int64_t n = (int64_t)2 * G * L.ny * L.nz;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int g = (int)(t % (2 * G));
        const int64_t jk = t / (2 * G);
        const int j = (int)(jk % L.ny), k = (int)(jk / L.ny);
        const int i = g < G ? g - G : L.nx + (g - G);
        const int per = g < G ? pm : pp;
        const int s = per ? ((i % L.nx) + L.nx) % L.nx : (i < 0 ? 0 : L.nx - 1);
        const int64_t d = L.at(i, j, k), o = L.at(s, j, k);
#pragma unroll
        for (int f = 0; f < NF3; ++f) S[d + f * fs] = S[o + f * fs];
    }
}

__global__ void k3_fill_y(double *S, int64_t fs, Layout3 L, int pm, int pp, const Dev3 *sc) {
    if (!sc->active) return;
    const int wx = L.nx + 2 * G;
    const int64_t n = (int64_t)2 * G * wx * L.nz;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t % wx) - G;
        const int64_t gk = t / wx;
        const int g = (int)(gk % (2 * G)), k = (int)(gk / (2 * G));
        const int j = g < G ? g - G : L.ny + (g - G);
        const int per = g < G ? pm : pp;
        const int s = per ? ((j % L.ny) + L.ny) % L.ny : (j < 0 ? 0 : L.ny - 1);
        const int64_t d = L.at(i, j, k), o = L.at(i, s, k);
#pragma unroll
        for (int f = 0; f < NF3; ++f) S[d + f * fs] = S[o + f * fs];
    }
}

__global__ void k3_fill_z(double *S, int64_t fs, Layout3 L, int pm, int pp, const Dev3 *sc) {
    if (!sc->active) return;
    const int wx = L.nx + 2 * G, wy = L.ny + 2 * G;
    const int64_t n = (int64_t)2 * G * wx * wy;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t % wx) - G;
        const int64_t r = t / wx;
        const int j = (int)(r % wy) - G;
        const int g = (int)(r / wy);
        const int k = g < G ? g - G : L.nz + (g - G);
        const int per = g < G ? pm : pp;
        const int s = per ? ((k % L.nz) + L.nz) % L.nz : (k < 0 ? 0 : L.nz - 1);
        const int64_t d = L.at(i, j, k), o = L.at(i, j, s);
#pragma unroll
        for (int f = 0; f < NF3; ++f) S[d + f * fs] = S[o + f * fs];
    }
}

struct Ptr8 {
    const double *p[NF3];
};
struct MPtr8 {
    double *p[NF3];
};

__global__ void k3_export(const double *U, int64_t fs, Layout3 L, MPtr8 dst, uint32_t mask, int64_t pitch,
                          int64_t ppitch) {
    const int64_t n = (int64_t)L.nx * L.ny * L.nz;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t % L.nx);
        const int64_t jk = t / L.nx;
        const int j = (int)(jk % L.ny), k = (int)(jk / L.ny);
        const int64_t s = L.at(i, j, k), d = i + j * pitch + k * ppitch;
#pragma unroll
        for (int f = 0; f < NF3; ++f)
            if (mask & (1u << f)) dst.p[f][d] = U[s + f * fs];
    }
}

// the caller's fields into the state, and in the same pass over them the
// state's wave speeds into slot 0 (as two passes 256^3 took 0.38 + 0.22 ms)
__global__ __launch_bounds__(256) void k3_import(double *U, int64_t fs, Layout3 L, Ptr8 src, int64_t pitch,
                                                 int64_t ppitch, double gamma, Dev3 *sc) {
    __shared__ double red[4][4];
    Speeds3 sp;
    const int64_t n = (int64_t)L.nx * L.ny * L.nz;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t % L.nx);
        const int64_t jk = t / L.nx;
        const int j = (int)(jk % L.ny), k = (int)(jk / L.ny);
        const int64_t d = L.at(i, j, k), o = i + j * pitch + k * ppitch;
        double u[NF3];
#pragma unroll
        for (int f = 0; f < NF3; ++f) u[f] = src.p[f][o];
#pragma unroll
        for (int f = 0; f < NF3; ++f) U[d + f * fs] = u[f];
        sp.add(u, gamma - 1.0, gamma);
    }
    sp.reduce(red, threadIdx.x >> 6, threadIdx.x & 63);
    __syncthreads();
    raise_speeds(red, sc, 0);
}

__global__ void k3_reset(Dev3 *sc, double t0) {
    memset(sc, 0, sizeof(Dev3));
    sc->t = t0;
    sc->active = 1;
}

// Between two steps: close the step that ran (`end`; not if it was switched
// off) and open the next (`begin`): its dt from the reduced wave speeds
// (minimum of h_d / c_d over the directions with more than one cell, taken x,
// y, z, then the end-time clamp) and the per-step constants.
// One wave, its loads issued at once, as for the 2-D scheme.
__global__ __launch_bounds__(64) void k3_step(Dev3 *sc, double t_end, Consts3 k, bool end, bool begin) {
    const int lane = threadIdx.x;
    const unsigned long long v = sacx::speeds_by_lane(sc->acc, lane);
    const int active = sc->active, cur0 = sc->cur, nonphys = sc->nonphys;
    const long long steps = sc->steps;
    const double dt0 = sc->dt, t0 = sc->t;
    end = end && active;
    const int cur = end ? cur0 ^ 1 : cur0;
    double c[3];
    for (int d = 0; d < 3; ++d) c[d] = __longlong_as_double((long long)__shfl(v, 32 * cur + d));
    if (begin) sacx::speeds_clear_by_lane(sc->acc[cur ^ 1], lane);
    if (lane) return;
    const double t = end ? t0 + dt0 : t0;
    if (end) {
        sc->t = t;
        sc->steps = steps + 1;
        sc->cur = cur;
    }
    if (!begin) return;
    sc->t_end = t_end;
    if (nonphys || (t_end > 0.0 && t_end - t <= 1e-12 * t_end)) { sc->active = 0; return; }
    double m = -1.0, cm = -1.0;
    for (int d = 0; d < 3; ++d) {
        if (!k.act[d]) continue;
        const double q = k.h[d] / c[d];
        m = m < 0.0 ? q : (m < q ? m : q);
        cm = cm < 0.0 ? c[d] : (cm > c[d] ? cm : c[d]);
    }
    double dt = k.cfl * m;
    if (t_end > 0.0) dt = (dt < t_end - t) ? dt : t_end - t;
    sc->dt = dt;
    sc->cmax = cm;
    for (int d = 0; d < 3; ++d) sc->last_c[d] = c[d];
    sc->last_cmax = cm;
    sc->hdt = 0.5 * dt;
    sc->dt6 = dt / 6.0;
    for (int d = 0; d < 3; ++d)
        for (int q = 0; q < 4; ++q) sc->kd2[d][q] = k.c2[q] * k.h[d] * cm;
    sc->active = 1;
}

// conservation sums: each block sums a contiguous run of cells (storage
// order) per field; the partials are added in block order
__global__ void k3_sums_partial(const double *U, int64_t fs, Layout3 L, double *part, int npart) {
    __shared__ double red[NF3][4];
    const int64_t n = (int64_t)L.nx * L.ny * L.nz;
    const int64_t per = (n + npart - 1) / npart;
    const int64_t b0 = blockIdx.x * per, b1 = min(n, b0 + per);
    double acc[NF3];
#pragma unroll
    for (int f = 0; f < NF3; ++f) acc[f] = 0.0;
    for (int64_t t = b0 + threadIdx.x; t < b1; t += blockDim.x) {
        const int i = (int)(t % L.nx);
        const int64_t jk = t / L.nx;
        const int j = (int)(jk % L.ny), k = (int)(jk / L.ny);
        const int64_t o = L.at(i, j, k);
#pragma unroll
        for (int f = 0; f < NF3; ++f) acc[f] += U[o + f * fs];
    }
#pragma unroll
    for (int f = 0; f < NF3; ++f)
        for (int off = 32; off > 0; off >>= 1) acc[f] += __shfl_down(acc[f], off);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int f = 0; f < NF3; ++f) red[f][w] = acc[f];
    __syncthreads();
    if (threadIdx.x < NF3) {
        double s = 0.0;
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += red[threadIdx.x][k];
        part[blockIdx.x * NF3 + threadIdx.x] = s;
    }
}

__global__ void k3_sums_final(const double *part, int npart, double *out, double cell) {
    const int f = threadIdx.x;
    if (f >= NF3) return;
    double s = 0.0;
    for (int b = 0; b < npart; ++b) s += part[b * NF3 + f];
    out[f] = s * cell;
}

struct Plan3 {
    Layout3 L;
    size_t field_bytes;
    size_t off_sc, off_part, off_sums, off_state, off_g, total;
};

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

int check3(const sacx3_grid *g, const sacx3_params *p) {
    using sacx::set_error;
    if (!g || !p) return set_error(SACX_EINVAL, "grid and params must not be NULL");
    if (g->nx < 1 || g->ny < 1 || g->nz < 1) return set_error(SACX_EINVAL, "nx, ny, nz must be >= 1");
    if ((int64_t)g->nx * g->ny * g->nz < 2) return set_error(SACX_EINVAL, "a grid needs more than one cell");
    if (g->nx > (1 << 20) || g->ny > (1 << 20) || g->nz > (1 << 20))
        return set_error(SACX_EINVAL, "a side exceeds 2^20 cells");
    if (!(g->x1 > g->x0) || !(g->y1 > g->y0) || !(g->z1 > g->z0) || !std::isfinite(g->x0) ||
        !std::isfinite(g->x1) || !std::isfinite(g->y0) || !std::isfinite(g->y1) || !std::isfinite(g->z0) ||
        !std::isfinite(g->z1))
        return set_error(SACX_EINVAL, "the extent must be finite with x1 > x0, y1 > y0, z1 > z0");
    if (!(p->gamma > 1.0) || !std::isfinite(p->gamma)) return set_error(SACX_EINVAL, "gamma must be > 1");
    if (!(p->cfl > 0.0) || !std::isfinite(p->cfl)) return set_error(SACX_EINVAL, "cfl must be > 0");
    for (int k = 0; k < 4; ++k)
        if (!(p->c2[k] >= 0.0) || !(p->cshk[k] >= 0.0) || !std::isfinite(p->c2[k]) || !std::isfinite(p->cshk[k]))
            return set_error(SACX_EINVAL, "hyper-diffusion constants must be finite and >= 0");
    // the kernels address a field array with 32-bit byte offsets
    const int64_t pitch = (int64_t)round_up((size_t)kAlign / sizeof(double) + g->nx + G, kAlign / sizeof(double));
    const double bytes = 8.0 * (double)pitch * (double)(g->ny + 2 * G) * (double)(g->nz + 2 * G);
    if (bytes > 4294967040.0)
        return set_error(SACX_EUNSUP, "one field array would take %.3g bytes; at most 4 GiB (about 800^3 cells)", bytes);
    return SACX_OK;
}

Plan3 plan3(const sacx3_grid *g, const sacx3_params *p) {
    Plan3 P;
    Layout3 &L = P.L;
    L.nx = g->nx; L.ny = g->ny; L.nz = g->nz;
    L.xoff = kAlign / (int)sizeof(double);
    L.pitch = (int)round_up((size_t)L.xoff + L.nx + G, kAlign / sizeof(double));
    L.plane = (int64_t)L.pitch * (L.ny + 2 * G);
    L.field_elems = (int64_t)round_up((size_t)(L.plane * (L.nz + 2 * G)), kAlign / sizeof(double));
    P.field_bytes = (size_t)L.field_elems * sizeof(double);
    size_t o = 0;
    P.off_sc = o; o = round_up(o + sizeof(Dev3), kAlign);
    P.off_part = o; o = round_up(o + sizeof(double) * NF3 * kPartials, kAlign);
    P.off_sums = o; o = round_up(o + sizeof(double) * NF3, kAlign);
    P.off_state = o; o += 4 * NF3 * P.field_bytes;
    P.off_g = o; o += p->hd_on ? 3 * NQF * P.field_bytes : 0;
    P.total = o;
    return P;
}

struct DevGuard {
    int prev = -1;
    bool ok = false;
    explicit DevGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) return;
        ok = prev == dev || hipSetDevice(dev) == hipSuccess;
    }
    ~DevGuard() {
        if (ok && prev >= 0) (void)hipSetDevice(prev);
    }
};

}  // namespace sacx3i

using namespace sacx3i;

struct sacx3_ctx {
    sacx3_grid grid;
    sacx3_params params;
    int device;
    hipStream_t stream;
    Plan3 P;
    char *ws;
    Dev3 *sc;
    double *part, *sums;
    double *U, *B1, *B2, *A, *Gf;
    int64_t fs;
    Consts3 kc;
    int bc[6];
    int tz, tzf;       // planes per block of the stage and the face launch
    bool initialized;
};

namespace sacx3i {

#define HIPCHK3(expr)                                                                                      \
    do {                                                                                                   \
        hipError_t e_ = (expr);                                                                            \
        if (e_ != hipSuccess)                                                                              \
            return sacx::set_error(SACX_EDEVICE, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, \
                                   __LINE__);                                                              \
    } while (0)

int blocks_for(int64_t n, int nt) {
    int64_t b = (n + nt - 1) / nt;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, 65536));
}

// Planes per block of one launch: every block marches its strip of planes
// after `warm` warm-up planes, so a launch takes about rounds x (strip +
// warm) planes, rounds = blocks / resident blocks rounded up.  The strip
// count that minimises this, of strips of at most 64 planes; 64 unless that
// gains more than 5 %.  Longer strips save warm-up planes and lose the overlap
// of neighbouring tiles in L2: the face launch takes 11.65 ms at 512^3 with 64
// planes and 12.30 with 129, a step 97.8 and 101.1.
// At 75 x 53 x 61 strips of 64 planes are 21 blocks on 256 compute units.
int planes_for(int64_t columns, int nz, int64_t slots, int warm) {
    auto cost = [&](int64_t tz) {
        const int64_t nb = columns * ((nz + tz - 1) / tz);
        return (double)((nb + slots - 1) / slots) * (double)(std::min<int64_t>(tz, nz) + warm);
    };
    int best = 64;
    double c = 0.95 * cost(64);
    for (int strips = 1; strips <= nz; ++strips) {
        const int tz = (nz + strips - 1) / strips;
        if (tz > 64) continue;
        if (cost(tz) < c) { c = cost(tz); best = tz; }
        if (columns * strips > 8 * slots) break;
    }
    return best;
}

void auto_planes(sacx3_ctx *c) {
    int cus = 0, per = 0, perf = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device);
    if (e == hipSuccess)
        e = c->params.hd_on ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k3_stage_hd<1, TXF, TYF>, 2 * NT, 0)
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k3_stage<1, TXF, TYF>, NT, 0);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&perf, k3_faces<TXF, TYF>, NT, 0);
    if (e != hipSuccess || cus < 1 || per < 1 || perf < 1) {
        (void)hipGetLastError();
        cus = 256;
        per = 1;
        perf = 2;
    }
    const Layout3 &L = c->P.L;
    auto tiles = [](int n, int t) { return (int64_t)((n + t - 1) / t); };
    c->tz = planes_for(tiles(L.nx, TXF) * tiles(L.ny, TYF), L.nz, (int64_t)cus * per, 2);
    c->tzf = planes_for(tiles(L.nx + 2, TXF) * tiles(L.ny + 2, TYF), L.nz + 2, (int64_t)cus * perf, 5);
}

// The launches read the cells outside through the maps, which replaces three
// fill launches per stage (256^3: 54, 14 and 13 us per stage).  A map shifts
// a periodic position by one period, so a periodic direction of fewer than G
// cells keeps filled ghost layers, all of them, and maps that leave positions
// in the ghost layers as they are.
bool narrow(const sacx3_ctx *c) {
    const Layout3 &L = c->P.L;
    const int n[3] = {L.nx, L.ny, L.nz};
    for (int d = 0; d < 3; ++d)
        if (n[d] < G && c->bc[2 * d] == SACX_PERIODIC) return true;
    return false;
}

void side_maps(const sacx3_ctx *c, SideMap (&m)[3]) {
    const Layout3 &L = c->P.L;
    const int n[3] = {L.nx, L.ny, L.nz};
    for (int d = 0; d < 3; ++d) {
        m[d] = sacx::side_map(n[d], c->bc[2 * d], c->bc[2 * d + 1]);
        if (narrow(c)) {
            m[d].lo = -G;
            m[d].hi = n[d] + G - 1;
            m[d].below = m[d].above = 0;
        }
    }
}

int fill3(sacx3_ctx *c, double *S) {
    const Layout3 &L = c->P.L;
    const int nt = 256;
    hipLaunchKernelGGL(k3_fill_x, dim3(blocks_for((int64_t)2 * G * L.ny * L.nz, nt)), dim3(nt), 0, c->stream, S,
                       c->fs, L, c->bc[0] == SACX_PERIODIC, c->bc[1] == SACX_PERIODIC, c->sc);
    hipLaunchKernelGGL(k3_fill_y, dim3(blocks_for((int64_t)2 * G * (L.nx + 2 * G) * L.nz, nt)), dim3(nt), 0,
                       c->stream, S, c->fs, L, c->bc[2] == SACX_PERIODIC, c->bc[3] == SACX_PERIODIC, c->sc);
    hipLaunchKernelGGL(k3_fill_z, dim3(blocks_for((int64_t)2 * G * (L.nx + 2 * G) * (L.ny + 2 * G), nt)), dim3(nt),
                       0, c->stream, S, c->fs, L, c->bc[4] == SACX_PERIODIC, c->bc[5] == SACX_PERIODIC, c->sc);
    HIPCHK3(hipGetLastError());
    return SACX_OK;
}

template <int STAGE>
int launch_stage3(sacx3_ctx *c, const Stage3Args &a, int nblocks) {
    if (c->params.hd_on)
        hipLaunchKernelGGL((k3_stage_hd<STAGE, TXF, TYF>), dim3(nblocks), dim3(2 * NT), 0, c->stream, a);
    else
        hipLaunchKernelGGL((k3_stage<STAGE, TXF, TYF>), dim3(nblocks), dim3(NT), 0, c->stream, a);
    HIPCHK3(hipGetLastError());
    return SACX_OK;
}

int stage3(sacx3_ctx *c, int s, double *S, double *U, double *A, double *o1, double *o2) {
    const Layout3 &L = c->P.L;
    if (narrow(c)) {
        int rc = fill3(c, S);
        if (rc) return rc;
    }
    SideMap m[3];
    side_maps(c, m);
    if (c->params.hd_on) {
        Face3Args f;
        f.mx = m[0]; f.my = m[1]; f.mz = m[2];
        f.S = S; f.Gf = c->Gf; f.fs = c->fs; f.L = L; f.k = c->kc; f.sc = c->sc; f.tz = c->tzf;
        f.ntx = (L.nx + 2 + TXF - 1) / TXF;
        f.nty = (L.ny + 2 + TYF - 1) / TYF;
        const int nzs = (L.nz + 2 + c->tzf - 1) / c->tzf;
        hipLaunchKernelGGL((k3_faces<TXF, TYF>), dim3(f.ntx * f.nty * nzs), dim3(NT), 0, c->stream, f);
        HIPCHK3(hipGetLastError());
    }
    Stage3Args a;
    a.mx = m[0]; a.my = m[1]; a.mz = m[2];
    a.S = S; a.U = U; a.A = A; a.out1 = o1; a.out2 = o2; a.Gf = c->Gf; a.fs = c->fs; a.L = L; a.k = c->kc;
    a.sc = c->sc; a.tz = c->tz; a.cross = c->params.hd_cross_on;
    a.ntx = (L.nx + TXF - 1) / TXF;
    a.nty = (L.ny + TYF - 1) / TYF;
    const int nb = a.ntx * a.nty * ((L.nz + c->tz - 1) / c->tz);
    switch (s) {
        case 1: return launch_stage3<1>(c, a, nb);
        case 2: return launch_stage3<2>(c, a, nb);
        case 3: return launch_stage3<3>(c, a, nb);
        default: return launch_stage3<4>(c, a, nb);
    }
}

}  // namespace sacx3i

#define fail sacx::set_error

extern "C" {

int sacx3_workspace_size(const sacx3_grid *grid, const sacx3_params *params, size_t *bytes) {
    if (!bytes) return fail(SACX_EINVAL, "bytes must not be NULL");
    int rc = check3(grid, params);
    if (rc) return rc;
    *bytes = plan3(grid, params).total;
    return SACX_OK;
}

int sacx3_create(const sacx3_grid *grid, const sacx3_params *params, void *d_ws, size_t ws_bytes, void *hip_stream,
                 sacx3_ctx **out) {
    if (!out) return fail(SACX_EINVAL, "out must not be NULL");
    *out = nullptr;
    int rc = check3(grid, params);
    if (rc) return rc;
    if (!d_ws) return fail(SACX_EINVAL, "d_ws must not be NULL");
    if ((uintptr_t)d_ws % kAlign) return fail(SACX_EINVAL, "d_ws must be 256-byte aligned");
    const Plan3 P = plan3(grid, params);
    if (ws_bytes < P.total) return fail(SACX_ENOSPC, "workspace of %zu bytes, %zu needed", ws_bytes, P.total);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(SACX_EDEVICE, "no current device");
    sacx3_ctx *c = new (std::nothrow) sacx3_ctx();
    if (!c) return fail(SACX_EINVAL, "out of host memory");
    c->grid = *grid;
    c->params = *params;
    c->device = dev;
    c->stream = (hipStream_t)hip_stream;
    c->P = P;
    c->ws = (char *)d_ws;
    c->sc = (Dev3 *)(c->ws + P.off_sc);
    c->part = (double *)(c->ws + P.off_part);
    c->sums = (double *)(c->ws + P.off_sums);
    c->fs = P.L.field_elems;
    const size_t blk = (size_t)NF3 * P.field_bytes;
    c->U = (double *)(c->ws + P.off_state);
    c->B1 = (double *)(c->ws + P.off_state + blk);
    c->B2 = (double *)(c->ws + P.off_state + 2 * blk);
    c->A = (double *)(c->ws + P.off_state + 3 * blk);
    c->Gf = params->hd_on ? (double *)(c->ws + P.off_g) : nullptr;
    for (int s = 0; s < 6; ++s) c->bc[s] = SACX_PERIODIC;
    auto_planes(c);
    // constants of the scheme (FP64, once)
    Consts3 &k = c->kc;
    memset(&k, 0, sizeof(k));
    const double ext[3][2] = {{grid->x0, grid->x1}, {grid->y0, grid->y1}, {grid->z0, grid->z1}};
    const int n[3] = {grid->nx, grid->ny, grid->nz};
    k.gamma = params->gamma;
    k.gm1 = params->gamma - 1.0;
    k.igm1 = 1.0 / k.gm1;
    k.third = 1.0 / 3.0;
    k.cfl = params->cfl;
    for (int q = 0; q < 4; ++q) k.c2[q] = params->c2[q];
    for (int d = 0; d < 3; ++d) {
        const double h = (ext[d][1] - ext[d][0]) / n[d];
        k.h[d] = h;
        k.ih[d] = 1.0 / h;
        k.i12[d] = 1.0 / (12.0 * h);
        k.i2[d] = 1.0 / (2.0 * h);
        for (int q = 0; q < 4; ++q) k.kds[d][q] = params->cshk[q] * h * h;
        k.act[d] = n[d] > 1;
    }
    c->initialized = false;
    *out = c;
    return SACX_OK;
}

int sacx3_destroy(sacx3_ctx *ctx) {
    if (!ctx) return SACX_OK;
    int rc = SACX_OK;
    {
        DevGuard dg(ctx->device);
        if (dg.ok && hipStreamSynchronize(ctx->stream) != hipSuccess)
            rc = fail(SACX_EDEVICE, "waiting for the context's stream failed");
    }
    delete ctx;
    return rc;
}

int sacx3_set_boundaries(sacx3_ctx *ctx, const int32_t bc[6]) {
    if (!ctx || !bc) return fail(SACX_EINVAL, "ctx and bc must not be NULL");
    const int n[3] = {ctx->grid.nx, ctx->grid.ny, ctx->grid.nz};
    for (int s = 0; s < 6; ++s)
        if (bc[s] != SACX_PERIODIC && bc[s] != SACX_OPEN) return fail(SACX_EINVAL, "side %d: unknown boundary %d", s, bc[s]);
    for (int d = 0; d < 3; ++d) {
        if ((bc[2 * d] == SACX_PERIODIC) != (bc[2 * d + 1] == SACX_PERIODIC))
            return fail(SACX_EINVAL, "direction %d: periodic sides must come in pairs", d);
        if (n[d] == 1 && bc[2 * d] != SACX_PERIODIC)
            return fail(SACX_EINVAL, "direction %d has one cell and must be periodic", d);
    }
    for (int s = 0; s < 6; ++s) ctx->bc[s] = bc[s];
    return SACX_OK;
}

int sacx3_set_launch(sacx3_ctx *ctx, int32_t planes) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (planes < 0 || planes > 4096) return fail(SACX_EINVAL, "planes must be in [0, 4096]");
    if (planes == 0) {
        DevGuard dg(ctx->device);
        auto_planes(ctx);
    } else {
        ctx->tz = ctx->tzf = planes;
    }
    return SACX_OK;
}

int sacx3_init_state(sacx3_ctx *ctx, const double *const *d_fields, int64_t pitch, int64_t plane_pitch, double t0) {
    if (!ctx || !d_fields) return fail(SACX_EINVAL, "ctx and d_fields must not be NULL");
    for (int f = 0; f < NF3; ++f)
        if (!d_fields[f]) return fail(SACX_EINVAL, "field %d pointer is NULL", f);
    if (pitch < ctx->grid.nx || plane_pitch < pitch * ctx->grid.ny)
        return fail(SACX_EINVAL, "pitch must be >= nx and plane_pitch >= ny * pitch");
    if (!std::isfinite(t0)) return fail(SACX_EINVAL, "t0 must be finite");
    DevGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const Layout3 &L = ctx->P.L;
    Ptr8 src;
    for (int f = 0; f < NF3; ++f) src.p[f] = d_fields[f];
    const int64_t ncell = (int64_t)L.nx * L.ny * L.nz;
    hipLaunchKernelGGL(k3_reset, dim3(1), dim3(1), 0, ctx->stream, ctx->sc, t0);
    hipLaunchKernelGGL(k3_import, dim3(std::min(blocks_for(ncell, 256), 8192)), dim3(256), 0, ctx->stream, ctx->U,
                       ctx->fs, L, src, pitch, plane_pitch, ctx->kc.gamma, ctx->sc);
    HIPCHK3(hipGetLastError());
    ctx->initialized = true;
    return SACX_OK;
}

int sacx3_advance(sacx3_ctx *ctx, int32_t nsteps, double t_end, int32_t *steps_done, double *t_now) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (nsteps < 0) return fail(SACX_EINVAL, "nsteps must be >= 0");
    if (!std::isfinite(t_end)) return fail(SACX_EINVAL, "t_end must be finite");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx3_init_state has not been called");
    DevGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const bool sync = steps_done || t_now;
    long long steps0 = 0;
    if (sync) {
        HIPCHK3(hipMemcpyAsync(&steps0, &ctx->sc->steps, sizeof(steps0), hipMemcpyDeviceToHost, ctx->stream));
        HIPCHK3(hipStreamSynchronize(ctx->stream));
    }
    const int chunk = sync ? 64 : (nsteps > 0 ? nsteps : 1);
    for (int n0 = 0; n0 < nsteps; n0 += chunk) {
        const int n1 = std::min(nsteps, n0 + chunk);
        for (int n = n0; n < n1; ++n) {
            hipLaunchKernelGGL(k3_step, dim3(1), dim3(64), 0, ctx->stream, ctx->sc, t_end, ctx->kc, n > n0, true);
            int rc;
            if ((rc = stage3(ctx, 1, ctx->U, nullptr, nullptr, ctx->B1, nullptr))) return rc;
            if ((rc = stage3(ctx, 2, ctx->B1, ctx->U, nullptr, ctx->B2, ctx->A))) return rc;
            if ((rc = stage3(ctx, 3, ctx->B2, ctx->U, nullptr, ctx->B1, nullptr))) return rc;
            if ((rc = stage3(ctx, 4, ctx->B1, nullptr, ctx->A, ctx->U, nullptr))) return rc;
            HIPCHK3(hipGetLastError());
        }
        hipLaunchKernelGGL(k3_step, dim3(1), dim3(64), 0, ctx->stream, ctx->sc, t_end, ctx->kc, true, false);
        HIPCHK3(hipGetLastError());
        if (sync && n1 < nsteps) {
            int act = 1;
            HIPCHK3(hipMemcpyAsync(&act, &ctx->sc->active, sizeof(act), hipMemcpyDeviceToHost, ctx->stream));
            HIPCHK3(hipStreamSynchronize(ctx->stream));
            if (!act) break;
        }
    }
    if (sync) {
        Dev3 h;
        HIPCHK3(hipMemcpyAsync(&h, ctx->sc, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
        HIPCHK3(hipStreamSynchronize(ctx->stream));
        if (steps_done) *steps_done = (int32_t)(h.steps - steps0);
        if (t_now) *t_now = h.t;
        if (h.nonphys) return fail(SACX_ENONPHYS, "non-physical state after %lld steps", h.steps);
    }
    return SACX_OK;
}

int sacx3_read_fields(sacx3_ctx *ctx, double *const *d_out, int64_t pitch, int64_t plane_pitch, uint32_t field_mask) {
    if (!ctx || !d_out) return fail(SACX_EINVAL, "ctx and d_out must not be NULL");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx3_init_state has not been called");
    if (pitch < ctx->grid.nx || plane_pitch < pitch * ctx->grid.ny)
        return fail(SACX_EINVAL, "pitch must be >= nx and plane_pitch >= ny * pitch");
    if (field_mask & ~0xFFu) return fail(SACX_EINVAL, "field_mask has bits beyond the 8 fields");
    MPtr8 dst;
    for (int f = 0; f < NF3; ++f) {
        dst.p[f] = (field_mask & (1u << f)) ? d_out[f] : nullptr;
        if ((field_mask & (1u << f)) && !d_out[f]) return fail(SACX_EINVAL, "output %d pointer is NULL", f);
    }
    DevGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const Layout3 &L = ctx->P.L;
    hipLaunchKernelGGL(k3_export, dim3(blocks_for((int64_t)L.nx * L.ny * L.nz, 256)), dim3(256), 0, ctx->stream,
                       ctx->U, ctx->fs, L, dst, field_mask, pitch, plane_pitch);
    HIPCHK3(hipGetLastError());
    return SACX_OK;
}

int sacx3_diagnostics(sacx3_ctx *ctx, sacx3_diag *out) {
    if (!ctx || !out) return fail(SACX_EINVAL, "ctx and out must not be NULL");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx3_init_state has not been called");
    DevGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const Layout3 &L = ctx->P.L;
    const int64_t n = (int64_t)L.nx * L.ny * L.nz;
    const int npart = (int)std::max<int64_t>(1, std::min<int64_t>(kPartials, (n + 255) / 256));
    hipLaunchKernelGGL(k3_sums_partial, dim3(npart), dim3(256), 0, ctx->stream, ctx->U, ctx->fs, L, ctx->part, npart);
    const double cell = (ctx->kc.h[0] * ctx->kc.h[1]) * ctx->kc.h[2];
    hipLaunchKernelGGL(k3_sums_final, dim3(1), dim3(64), 0, ctx->stream, ctx->part, npart, ctx->sums, cell);
    HIPCHK3(hipGetLastError());
    Dev3 h;
    double sums[NF3];
    HIPCHK3(hipMemcpyAsync(&h, ctx->sc, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK3(hipMemcpyAsync(sums, ctx->sums, sizeof(sums), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK3(hipStreamSynchronize(ctx->stream));
    out->t = h.t;
    out->dt = h.dt;
    double c[3], cm = -1.0;
    for (int d = 0; d < 3; ++d) {
        const unsigned long long bits = sacx::speed_max(h.acc[h.cur], d);
        memcpy(&c[d], &bits, sizeof(double));
        out->c[d] = c[d];
        if (ctx->kc.act[d]) cm = cm < 0.0 ? c[d] : std::max(cm, c[d]);
    }
    out->c_max = cm;
    for (int f = 0; f < NF3; ++f) out->sums[f] = sums[f];
    out->steps = h.steps;
    out->nonphys = h.nonphys;
    return SACX_OK;
}

}  // extern "C"
