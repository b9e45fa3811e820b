// sacx_runtime.hip -- host runtime and C ABI of libsacx, plus the small
// auxiliary kernels (halo exchange, boundary fills, reductions, step scalars,
// field import/export).
//
// Time stepping (paper section 2, classic RK4) uses four state buffers U, B1,
// B2, A and the stage kernel's fused combine:
//   stage 1: B1 = U  + dt/2 L(U)
//   stage 2: B2 = U  + dt/2 L(B1),   A = 2U + ((B1 - U) + dt L(B1))
//   stage 3: B1 = U  + dt   L(B2)
//   stage 4: U  = B1 + (A - 2 B1)/3 + dt/6 L(B1)
// which is algebraically U + dt/6 (K1 + 2 K2 + 2 K3 + K4), leaves a state
// with L = 0 bit-for-bit unchanged, and moves 12 field values per cell and
// step (stencil reads 4, pointwise reads 3, writes 5).
//
// Cells beyond a periodic or an open side are read where the boundary has
// their values (SideMap), by the stage kernels themselves.  Ghost layers are
// filled only for exchange sides (paper section 3, exchange_halo: the
// domain's hand-over between subdomains, x first, then y over the padded
// width, so the corners travel), for periodic directions of fewer than 3
// cells, and for the stage-level calls, whose stages read the ghost cells that
// the caller completed.
//
// A call's steps take, by what is expected to be fastest, one launch per stage
// (marching strips or boxes), one per two stages (without hyper-diffusion) or
// one per step (tubes); the results are the same bits.
//
// The time step is computed on the device: stage 4 reduces max(|v_d| + c_f)
// of the new state into the next slot of a double-buffered accumulator, and
// one small launch between two steps advances t and turns the maxima into the
// next dt (with the end-time clamp).  Nothing synchronises with the host inside
// sacx_advance.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstdarg>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <exception>
#include <new>
#include <string>
#include <array>
#include <vector>

#include "sacx_internal.h"

using namespace sacx;

// ------------------------------------------------------------------ errors

static thread_local std::string g_last_error;

int sacx::set_error(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}
#define fail sacx::set_error

// work that allocates host memory, for an entry point that no exception may leave
template <typename F>
static int allocating(F &&work) {
    try {
        return work();
    } catch (const std::exception &e) {   // bad_alloc, or a vector's length_error
        return fail(SACX_EINVAL, "out of host memory (%s)", e.what());
    }
}


// ------------------------------------------------------------------ context

// a launch group between two events of a context's pool; class 0..3 = stage
// kernels, 4 = halo, 5 = scalar kernels, 6 = surrogate refresh; share: the part
// of its time that is the context's own
struct ProfMark {
    int cls, start, stop;
    double share;
};

struct sacx_ctx {
    sacx_grid grid;
    sacx_params params;
    int device;
    hipStream_t stream;
    Layout L;
    size_t elem;
    int bc[4];
    char *ws;
    size_t ws_bytes;
    DevScalars *sc;
    double *sums;      // 6 doubles
    int *unfilled;     // 1 while the ghost cells of a loaded state are not filled
    double *partials;  // npart x 6
    int npart;
    void *U[NF], *B1[NF], *B2[NF], *A[NF], *BG[NBG];
    void *hx[2], *hy[2];
    bool initialized;
    int ty, nt;
    int split;         // FP64 hyper-diffusion tiles: two threads per column
    int box;           // rows of the box kernel's blocks (4, 8, 16); 0: the marching kernels
    int cus;                // compute units of the device
    int pair_rows;          // rows per block of the two-stage kernel
    bool nt_auto, ty_auto;  // columns / strip height chosen by auto_rows (until set explicitly)
    double dx, dy;
    SchemeConsts kc;
    // profiling: event pairs recorded around launch groups, resolved at read
    bool prof_on;
    std::vector<hipEvent_t> *ev_pool;
    std::vector<ProfMark> *ev_marks;
    int ev_used;
    int prof_start;    // the start event of a launch group shared with other contexts
    sacx_profile prof;
    // learned hyper-diffusion coefficient (off unless sacx_hd_set_surrogate)
    bool sur_on;
    sacx_surrogate sur;
    float *sur_r;          // ratio planes
    unsigned char *sur_k;  // per check tile: prediction kept (1) or fallen back (0)
    int64_t sur_pitch;
    void *sur_x, *sur_a1, *sur_a2;
    HdDevStats *sur_st;
    int64_t sur_since;     // steps enqueued since the last refresh
    int64_t sur_refreshes, sur_tiles_checked;
    // decomposed stepping (sacx_stage): the next RK4 stage, 0 between steps
    int stage_next;
    // the ghost cells of a loaded state, and of the background, may still have
    // to be filled for the stage-level calls (the library's own steps read
    // through the maps)
    bool ghosts_due, bg_due;
    // bumped by every change a batch's instance table copies (boundaries,
    // spacing), so that the batch rebuilds its table
    unsigned long long gen;
};

namespace {

constexpr size_t kAlign = 256;
constexpr int kPartials = 512;

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Plan {
    Layout L;
    size_t elem;
    size_t field_bytes;
    size_t off_sc, off_sums, off_part, off_state, off_bg, off_hx, off_hy, total;
    size_t hx_bytes, hy_bytes;
};

int check_grid(const sacx_grid *g, const sacx_params *p) {
    if (!g || !p) return fail(SACX_EINVAL, "grid/params must not be NULL");
    if (g->nx < 1 || g->ny < 1) return fail(SACX_EINVAL, "nx, ny must be >= 1 (got %d, %d)", g->nx, g->ny);
    if (g->nx < 2 && g->ny < 2) return fail(SACX_EINVAL, "at least one direction needs 2 or more cells");
    if ((int64_t)g->nx * g->ny > ((int64_t)1 << 34)) return fail(SACX_EINVAL, "grid too large");
    if (g->nx > (1 << 24) || g->ny > (1 << 24)) return fail(SACX_EINVAL, "grid dimension too large");
    if (!(g->x1 > g->x0) || !(g->y1 > g->y0)) return fail(SACX_EINVAL, "empty physical extent");
    if (g->precision != SACX_FP64 && g->precision != SACX_FP32)
        return fail(SACX_EINVAL, "precision must be SACX_FP64 or SACX_FP32");
    if (g->background_on != 0 && g->background_on != 1) return fail(SACX_EINVAL, "background_on must be 0 or 1");
    if (!(p->gamma > 1.0) || !std::isfinite(p->gamma)) return fail(SACX_EINVAL, "gamma must be > 1");
    if (!(p->cfl > 0.0) || !std::isfinite(p->cfl)) return fail(SACX_EINVAL, "cfl must be > 0");
    for (int k = 0; k < 4; ++k)
        if (!(p->c2[k] >= 0.0) || !(p->cshk[k] >= 0.0) || !std::isfinite(p->c2[k]) || !std::isfinite(p->cshk[k]))
            return fail(SACX_EINVAL, "hyper-diffusion constants must be finite and >= 0");
    if (!std::isfinite(p->g[0]) || !std::isfinite(p->g[1])) return fail(SACX_EINVAL, "gravity must be finite");
    return SACX_OK;
}

Plan make_plan(const sacx_grid *g) {
    Plan P;
    P.elem = g->precision == SACX_FP64 ? 8 : 4;
    const int per = (int)(kAlign / P.elem);
    P.L.nx = g->nx;
    P.L.ny = g->ny;
    P.L.xoff = per;
    P.L.pitch = (int)round_up((size_t)per + g->nx + G, (size_t)per);
    P.L.rows = g->ny + 2 * G;
    P.L.field_elems = (int64_t)P.L.rows * P.L.pitch;
    P.field_bytes = round_up((size_t)P.L.field_elems * P.elem, kAlign);
    size_t off = 0;
    P.off_sc = off; off += round_up(sizeof(DevScalars), kAlign);
    P.off_sums = off; off += kAlign;
    P.off_part = off; off += round_up((size_t)kPartials * NF * sizeof(double), kAlign);
    P.off_state = off; off += 4 * NF * P.field_bytes;
    P.off_bg = off; off += g->background_on ? NBG * P.field_bytes : 0;
    P.hx_bytes = round_up((size_t)NF * G * g->ny * P.elem, kAlign);
    P.hy_bytes = round_up((size_t)NF * G * (g->nx + 2 * G) * P.elem, kAlign);
    P.off_hx = off; off += 2 * P.hx_bytes;
    P.off_hy = off; off += 2 * P.hy_bytes;
    P.total = off;
    return P;
}

// Output rows per strip.  When the whole grid fits in one round of resident
// blocks (slots) with strips of at most 512 rows, the strip count whose
// longest block (strip plus the 6-row warm-up) is shortest; otherwise strips
// of 256 rows, halved while the launch has fewer than 1024 blocks.  (Measured
// on MI355X: FP32 at 8000^2 and FP64 at 2048^2 fit one round and gain from
// balanced strips; FP64 at 8000^2 takes several rounds and, being partly
// bandwidth-bound, runs a part-filled last round faster than a full one, so
// rounding the block count gains nothing there; the FP64 kernel without
// hyper-diffusion loses 6 % with one round of 534-row strips.)
int rows_for_slots(const Layout &L, int nt, int64_t slots) {
    if (L.ny <= 8) return L.ny;
    const int64_t xt = (L.nx + nt - 2 * G - 1) / (nt - 2 * G);
    int one = 0;
    for (int64_t strips = (L.ny + 4095) / 4096; strips <= (L.ny + 7) / 8; ++strips) {
        const int64_t ty = (L.ny + strips - 1) / strips;
        if (ty < 8) break;
        if (xt * ((L.ny + ty - 1) / ty) <= slots) one = (int)ty;   // later strips are shorter
        else break;
    }
    if (one > 0 && one <= 512) return one;
    int ty = 256;
    while (ty > 8 && xt * ((L.ny + ty - 1) / ty) < 1024) ty /= 2;
    return ty;
}

// Time per row of a block with 1, 2, ... blocks on its compute unit, in us
// (MI355X, the mean of the four stages, 24-row strips whose state stays in
// the caches; the third of the first row raised by what 1024^2 shows), by kernel
// and columns per block (64, 128, 256; 0: not
// measured, the last value stands).
enum { KIND_SPLIT = 0, KIND_SPLIT_BG, KIND_F64_NOHD, KIND_F32, KIND_F32_NOHD, KINDS };
const float kRowUs[KINDS][3][8] = {
    {{1.44f, 2.08f, 2.35f, 2.67f}, {1.66f, 2.68f}, {3.1f}},
    {{1.69f, 2.54f, 3.02f, 3.56f}, {2.10f, 3.54f}, {4.0f}},
    {{0.85f, 1.10f, 1.20f, 1.45f, 2.40f, 3.10f}, {1.07f, 1.60f, 3.00f}, {3.0f}},
    {{1.67f, 1.69f, 1.70f, 1.70f, 1.95f, 2.20f, 2.36f, 2.52f}, {1.88f, 2.12f, 2.29f, 2.45f}, {1.99f, 2.56f}},
    {{0.75f, 0.80f, 0.83f, 0.94f, 1.05f, 1.15f, 1.40f, 1.67f}, {0.86f, 0.95f, 1.20f, 1.60f}, {0.95f, 1.57f}},
};

// the smallest strip height whose blocks are at most `blocks`
int rows_for_blocks(const Layout &L, int nt, int64_t blocks) {
    const int64_t xt = (L.nx + nt - 2 * G - 1) / (nt - 2 * G);
    const int64_t strips = blocks / xt;
    return strips < 1 ? INT32_MAX : (int)((L.ny + strips - 1) / strips);
}

// The launch shape where the grid fits in one round of resident blocks: for
// each width and each number k of blocks per compute unit, the strip height
// that gives every unit k blocks takes about rows + 9 row times (6 warm-up
// rows, and about 3 for the launch); the cheapest is taken.  Narrow blocks
// and short strips pay where wide ones leave units idle: FP64 at 300 x 136
// takes 75 us per step with 128 x 2 strips and 109 with 128 x 8 (51 blocks),
// at 512^2 137 against 158; FP32 at 300 x 136 72 against 117, at 2048^2 397
// against 431; 1501 x 997 without hyper-diffusion 196 against 253.  Strips
// above 160 rows keep the default width: there the widths differ by less than
// the spread of the figures above.
bool shape_for_slots(const sacx_ctx *c, int cus, int *nt, int *ty, double *cost_us) {
    const bool fp64 = c->grid.precision == SACX_FP64;
    const bool hd = c->params.hd_on != 0, bg = c->grid.background_on != 0;
    if (c->L.ny <= 8 || (fp64 && hd && !c->split)) return false;
    const int kind = fp64 ? (hd ? (bg ? KIND_SPLIT_BG : KIND_SPLIT) : KIND_F64_NOHD) : (hd ? KIND_F32 : KIND_F32_NOHD);
    double best = 0.0;
    bool found = false;
    for (int w = 0; w < (fp64 ? 2 : 3); ++w) {
        const int cols = 64 << w;
        int per = 0;
        const hipError_t e = fp64 ? stage_blocks_per_cu<double>(cols, hd, bg, true, &per)
                                  : stage_blocks_per_cu<float>(cols, hd, bg, true, &per);
        if (e != hipSuccess) { (void)hipGetLastError(); continue; }
        for (int k = 1; k <= std::min(per, 8); ++k) {
            const float us = kRowUs[kind][w][k - 1];
            if (us == 0.0f) break;
            const int rows = rows_for_blocks(c->L, cols, (int64_t)cus * k);
            if (rows > 160) continue;
            const double cost = us * (rows + 9.0);
            if (!found || cost < best) { found = true; best = cost; *nt = cols; *ty = rows; }
        }
    }
    *cost_us = best;
    return found;
}

// A stage by the box kernel with `tiles` blocks: about 3 us to launch, `one`
// for the first block of a compute unit, and `round` for every two blocks per
// unit past the first 0.6 of that (us, MI355X, mean of the four stages).
struct BoxTime {
    float one, round;
};
const BoxTime kBoxUs[2][2][2] = {
    // no hyper-diffusion            with: 8 rows, 16 rows
    {{{4.2f, 7.8f}, {0.0f, 0.0f}}, {{7.5f, 11.4f}, {0.0f, 0.0f}}},   // FP64
    {{{3.5f, 4.4f}, {0.0f, 0.0f}}, {{5.0f, 5.5f}, {6.2f, 9.9f}}},    // FP32
};

double box_us(const BoxTime &b, int64_t tiles, int cus) {
    return 3.0 + b.one + b.round * std::max(0.0, (double)tiles / (2.0 * cus) - 0.6);
}

// The box kernel's rows where it is expected to take less than 0.95 of
// `march_us` (the marching shape's expected time) over the given tile
// counts (8 rows, 16 rows); 0 where it is not.
int box_for(bool fp32, bool hd, int64_t tiles8, int64_t tiles16, int cus, double march_us) {
    double best = 0.95 * march_us;
    int rows = 0;
    for (int k = 0; k < (fp32 && hd ? 2 : 1); ++k) {
        const double us = box_us(kBoxUs[fp32][hd][k], k ? tiles16 : tiles8, cus);
        if (us < best) { best = us; rows = k ? 16 : 8; }
    }
    return rows;
}

// Two stages per launch: without hyper-diffusion (with it a stage reaches 3
// cells to each side and is not bound by memory), a background or exchange
// sides, in the automatic launch shape, on grids whose periodic images are
// one period away from 4 cells outside.  Faster at every size tried, 64^2
// (29 -> 21 us per step) to 4000^2 (2524 -> 1400).
bool stage_pairs(const sacx_ctx *c) {
    if (c->params.hd_on || c->grid.background_on || c->sur_on || !c->nt_auto || !c->ty_auto) return false;
    for (int k = 0; k < 4; ++k)
        if (c->bc[k] == SACX_EXCHANGE) return false;
    return c->L.nx >= 8 && c->L.ny >= 8;
}

// Rows per block of the two-stage kernel: 24 re-read and recompute less, 8 make
// more blocks.  A compute unit holds one block of 24 rows or two of 8; the time
// is the rounds of 24-row blocks against a round's time of 8-row blocks (0.72 of
// the other in FP64, 0.84 in FP32) times the mean of their whole rounds and
// their number in rounds (their last round ends early where it is part-filled).
// Over sizes from 64^2 to 4000^2 this takes the slower one by more than 2 % at 10
// of 178 in FP64 (12 % at 2000 x 500, at most 4 % elsewhere) and at 6 of 153 in
// FP32 (at most 4 %).  us per step with 8 and with 24 rows, FP64:
// 300 x 136 19, 27; 392 x 600 38, 32; 700 x 500 47, 55; 900 x 700 68, 67; 1000 x 800
// 83, 88; 1501 x 997 148, 150; 2000^2 387, 377; 4000^2 1493, 1369; FP32: 300 x 136
// 16, 19; 700 x 500 30, 32; 900 x 700 42, 39; 1501 x 997 78, 76; 4000^2 808, 728.
int pair_rows_for(const Layout &L, bool fp64, int cus) {
    const int64_t xt = (L.nx + 55) / 56, t8 = xt * ((L.ny + 7) / 8), t24 = xt * ((L.ny + 23) / 24);
    const double r8 = 0.5 * ((double)((t8 + 2 * cus - 1) / (2 * cus)) + (double)t8 / (2 * cus));
    const double r24 = (double)((t24 + cus - 1) / cus);
    return r24 < (fp64 ? 0.72 : 0.84) * r8 ? 24 : 8;
}

int64_t box_tiles(const Layout &L, int rows) { return (int64_t)((L.nx + 57) / 58) * ((L.ny + rows - 1) / rows); }

// the launch shape for the context's current settings: resident blocks from
// the device's compute units and the kernel's occupancy.  Measured on MI355X:
// larger grids are best with 128 columns in FP64 (OT 8000^2, also with a
// background at 4000^2) and 256 in FP32.
void auto_rows(sacx_ctx *c) {
    int cus = 0, per = 0;
    const bool fp64 = c->grid.precision == SACX_FP64;
    const bool hd = c->params.hd_on != 0, bg = c->grid.background_on != 0;
    c->box = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device);
    c->cus = e == hipSuccess && cus > 0 ? cus : 256;
    c->pair_rows = pair_rows_for(c->L, fp64, c->cus);
    if (c->nt_auto) {
        c->nt = fp64 ? 128 : 256;
        double us = 0.0;
        if (e == hipSuccess && cus >= 1 && shape_for_slots(c, cus, &c->nt, &c->ty, &us)) {
            if (!bg) c->box = box_for(!fp64, hd, box_tiles(c->L, 8), box_tiles(c->L, 16), cus, us);
            // FP64 with half the rows while that makes no more blocks than
            // compute units: a wave's work is issue-bound there and twice the
            // units share it (64^2 40.1 -> 36.1 us per step, 300 x 136
            // 43.1 -> 40.3; 400 x 200, with 350 blocks, 46.9 -> 51.0; FP32
            // 30.6 -> 30.6 and slower)
            if (c->box == 8 && fp64 && hd && box_tiles(c->L, 4) <= cus) c->box = 4;
            return;
        }
    }
    if (e == hipSuccess)
        e = fp64 ? stage_blocks_per_cu<double>(c->nt, hd, bg, c->split != 0, &per)
                 : stage_blocks_per_cu<float>(c->nt, hd, bg, c->split != 0, &per);
    if (e != hipSuccess || cus < 1 || per < 1) {
        (void)hipGetLastError();
        cus = 256;
        per = 2;
    }
    c->ty = rows_for_slots(c->L, c->nt, (int64_t)cus * per);
}

// ------------------------------------------------------------------ kernels

template <typename real>
struct FPtr {
    real *p[NF];
};

__device__ __forceinline__ int64_t eidx(const Layout &L, int i, int j) {
    return (int64_t)L.xoff + i + (int64_t)(j + G) * L.pitch;
}

__device__ __forceinline__ bool step_active(const DevScalars *sc) { return sc->active != 0; }

// x strips: buffer [f][g][j], j in [0, ny)
template <typename real>
__global__ void k_pack_x(FPtr<real> S, int nf, Layout L, real *b0, real *b1, int sides, const DevScalars *sc) {
    if (sc && !step_active(sc)) return;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    const int side = (sides == 2) ? (int)blockIdx.z : sides - 10;
    if (j >= L.ny || f >= nf) return;
    real *b = side == 0 ? b0 : b1;
    const int c0 = side == 0 ? 0 : L.nx - G;
#pragma unroll
    for (int g = 0; g < G; ++g) b[((int64_t)f * G + g) * L.ny + j] = S.p[f][eidx(L, c0 + g, j)];
}

template <typename real>
__global__ void k_unpack_x(FPtr<real> S, int nf, Layout L, const real *b0, const real *b1, int sides,
                           const DevScalars *sc) {
    if (sc && !step_active(sc)) return;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    const int side = (sides == 2) ? (int)blockIdx.z : sides - 10;
    if (j >= L.ny || f >= nf) return;
    const real *b = side == 0 ? b0 : b1;
    const int cg = side == 0 ? -G : L.nx;
#pragma unroll
    for (int g = 0; g < G; ++g) S.p[f][eidx(L, cg + g, j)] = b[((int64_t)f * G + g) * L.ny + j];
}

// y strips over the padded width: buffer [f][g][i + G], i in [-G, nx + G),
// cells outside x read as mx says
template <typename real>
__global__ void k_pack_y(FPtr<real> S, int nf, Layout L, SideMap mx, real *b0, real *b1, int sides,
                         const DevScalars *sc) {
    if (sc && !step_active(sc)) return;
    const int w = L.nx + 2 * G;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    const int side = (sides == 2) ? (int)blockIdx.z : sides - 10;
    if (i >= w || f >= nf) return;
    real *b = side == 0 ? b0 : b1;
    const int r0 = side == 0 ? 0 : L.ny - G;
#pragma unroll
    for (int g = 0; g < G; ++g) b[((int64_t)f * G + g) * w + i] = S.p[f][eidx(L, mx.at(i - G), r0 + g)];
}

template <typename real>
__global__ void k_unpack_y(FPtr<real> S, int nf, Layout L, const real *b0, const real *b1, int sides,
                           const DevScalars *sc) {
    if (sc && !step_active(sc)) return;
    const int w = L.nx + 2 * G;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    const int side = (sides == 2) ? (int)blockIdx.z : sides - 10;
    if (i >= w || f >= nf) return;
    const real *b = side == 0 ? b0 : b1;
    const int rg = side == 0 ? -G : L.ny;
#pragma unroll
    for (int g = 0; g < G; ++g) S.p[f][eidx(L, i - G, rg + g)] = b[((int64_t)f * G + g) * w + i];
}

// open (zero-gradient) or small-periodic (index modulo n) fills; bit 0 / 1 of
// `skip` leaves the low / high side alone (a side filled by the caller)
template <typename real>
__global__ void k_fill_x(FPtr<real> S, int nf, Layout L, int periodic, int skip, const DevScalars *sc) {
    if (sc && !step_active(sc)) return;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    if (j >= L.ny || f >= nf) return;
    for (int g = 1; g <= G; ++g) {
        int il = -g, ir = L.nx - 1 + g;
        int sl, sr;
        if (periodic) {
            sl = ((il % L.nx) + L.nx) % L.nx;
            sr = ir % L.nx;
        } else {
            sl = 0;
            sr = L.nx - 1;
        }
        if (!(skip & 1)) S.p[f][eidx(L, il, j)] = S.p[f][eidx(L, sl, j)];
        if (!(skip & 2)) S.p[f][eidx(L, ir, j)] = S.p[f][eidx(L, sr, j)];
    }
}

template <typename real>
__global__ void k_fill_y(FPtr<real> S, int nf, Layout L, int periodic, int skip, const DevScalars *sc) {
    if (sc && !step_active(sc)) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x - G;
    const int f = blockIdx.y;
    if (i >= L.nx + G || f >= nf) return;
    for (int g = 1; g <= G; ++g) {
        int jl = -g, jr = L.ny - 1 + g;
        int sl, sr;
        if (periodic) {
            sl = ((jl % L.ny) + L.ny) % L.ny;
            sr = jr % L.ny;
        } else {
            sl = 0;
            sr = L.ny - 1;
        }
        if (!(skip & 1)) S.p[f][eidx(L, i, jl)] = S.p[f][eidx(L, i, sl)];
        if (!(skip & 2)) S.p[f][eidx(L, i, jr)] = S.p[f][eidx(L, i, sr)];
    }
}

// The ghost cells of both directions in one launch, for any kinds of sides, as
// fills of x over the interior rows and then of y over the padded width leave
// them: beyond exchange sides they stay as they are.  With a flag only while
// that is set: a captured graph that has this launch must not fill a loaded
// state a second time, over what the caller completed between its replays.
template <typename real>
__global__ void k_fill_ghosts(FPtr<real> S, Layout L, int4 bc, const int *unfilled) {
    if (unfilled && !*unfilled) return;
    const int W = L.nx + 2 * G;
    const int64_t ny_part = (int64_t)2 * G * W, n = ny_part + (int64_t)2 * G * L.ny;
    const int f = blockIdx.y;
    // the cell that one beyond the sides of a direction images (beyond an exchange side itself)
    auto image = [](int i, int cells, int lo, int hi) {
        const int kind = i < 0 ? lo : hi;
        if ((i >= 0 && i < cells) || kind == SACX_EXCHANGE) return i;
        return kind == SACX_PERIODIC ? (i % cells + cells) % cells : (i < 0 ? 0 : cells - 1);
    };
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        int i, j;
        if (k < ny_part) {
            const int g = (int)(k / W);
            i = (int)(k % W) - G;
            j = g < G ? g - G : L.ny + g - G;
        } else {
            const int64_t k2 = k - ny_part;
            const int g = (int)(k2 % (2 * G));
            j = (int)(k2 / (2 * G));
            i = g < G ? g - G : L.nx + g - G;
        }
        const int si = image(i, L.nx, bc.x, bc.y), sj = image(j, L.ny, bc.z, bc.w);
        const bool outside = si < 0 || si >= L.nx;   // beyond an exchange side of x
        if (sj < 0 || sj >= L.ny || (outside && sj == j)) continue;
        S.p[f][eidx(L, i, j)] = S.p[f][eidx(L, si, sj)];
    }
}

__global__ void k_set_int(int *p, int v) { *p = v; }

// caller arrays <-> internal storage
template <typename T>
struct CPtr {
    const T *p[NF];
};
template <typename T>
struct MPtr {
    T *p[NF];
};

template <typename real, typename T>
__global__ void k_import(FPtr<real> D, CPtr<T> src, int nf, Layout L, int64_t pitch) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    if (i >= L.nx) return;
    for (int f = 0; f < nf; ++f) D.p[f][eidx(L, i, j)] = (real)src.p[f][(int64_t)j * pitch + i];
}

// the verification problems evaluated at the cell centres x0 + (i + 1/2) hx,
// y0 + (j + 1/2) hy (the operations in the order the conserved variables are
// defined: e = p/(gamma-1) + rho |v|^2/2 + |B|^2/2)
template <typename real>
__global__ void k_init_problem(FPtr<real> D, Layout L, int kind, double x0, double hx, double y0, double hy,
                               double mid, int along_y, double gamma, double p0, double p1) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    if (i >= L.nx) return;
    const double x = x0 + ((double)i + 0.5) * hx, y = y0 + ((double)j + 0.5) * hy;
    double rho, vx, vy, p, bx, by;
    if (kind == SACX_PROBLEM_ORSZAG_TANG) {
        const double pi = 3.141592653589793;   // the double nearest pi
        const double b0 = p0 / sqrt(4.0 * pi);
        rho = 25.0 / (36.0 * pi);
        p = 5.0 / (12.0 * pi);
        vx = -sin(y);
        vy = sin(x);
        bx = -b0 * sin(y);
        by = b0 * sin(2.0 * x);
    } else {
        const bool left = (along_y ? y : x) < mid;
        rho = left ? 1.0 * p0 : 0.125 * p1;
        p = left ? 1.0 * p0 : 0.1 * p1;
        vx = 0.0;
        vy = 0.0;
        const double bn = 0.75, bt = left ? 1.0 : -1.0;
        bx = along_y ? bt : bn;
        by = along_y ? bn : bt;
    }
    const double e = p / (gamma - 1.0) + 0.5 * rho * (vx * vx + vy * vy) + 0.5 * (bx * bx + by * by);
    const int64_t o = eidx(L, i, j);
    D.p[0][o] = (real)rho;
    D.p[1][o] = (real)(rho * vx);
    D.p[2][o] = (real)(rho * vy);
    D.p[3][o] = (real)e;
    D.p[4][o] = (real)bx;
    D.p[5][o] = (real)by;
}

template <typename real, typename T>
__global__ void k_export(FPtr<real> Sx, MPtr<T> dst, uint32_t mask, Layout L, int64_t pitch) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    if (i >= L.nx) return;
    for (int f = 0; f < NF; ++f)
        if (mask & (1u << f)) dst.p[f][(int64_t)j * pitch + i] = (T)Sx.p[f][eidx(L, i, j)];
}

// |v_d| + c_f of one cell raised into cx, cy; bad where it is non-physical
template <typename real>
__device__ __forceinline__ void cell_speeds(const real (&u)[NF], real rb, real eb, real bxb, real byb, real gam,
                                            real gm1, double &cx, double &cy, int &bad) {
    const real half = (real)0.5;
    const real rt = u[0], mx = u[1], my = u[2], et = u[3], bxt = u[4], byt = u[5];
    const real r = rb + rt;
    const real ir = (real)1 / r;
    const real ux = mx * ir, uy = my * ir;
    const real kin = half * (mx * ux + my * uy);
    const real bbd = bxb * bxt + byb * byt;
    const real bt2 = bxt * bxt + byt * byt;
    const real pkt = gm1 * (((et - kin) - bbd) - half * bt2);
    const real b2b = bxb * bxb + byb * byb;
    const real pkb = gm1 * (eb - half * b2b);
    const real pk = pkb + pkt;
    const real bx = bxb + bxt, by = byb + byt;
    const real cf = sqrt((gam * pk + (bx * bx + by * by)) * ir);
    const bool fin = isfinite(rt) && isfinite(mx) && isfinite(my) && isfinite(et) && isfinite(bxt) && isfinite(byt) &&
                     isfinite(cf);
    if (!(r > (real)0) || !(pk > (real)0) || !fin) {
        bad = 1;
        return;
    }
    cx = fmax(cx, (double)(fabs(ux) + cf));
    cy = fmax(cy, (double)(fabs(uy) + cf));
}

// the maxima of a block of 256 threads into accumulator slot `slot`
__device__ __forceinline__ void block_speeds(double cx, double cy, int bad, DevScalars *sc, int slot) {
    __shared__ double red[3][4];
    raise_speeds(cx, cy, bad, red, sc, slot);
}

// the caller's evolved fields into the state, and in the same pass over them
// the wave speeds of the state (background already in place) into slot 0
// (as two passes, 8000^2 in FP64 took 1.09 + 0.67 ms)
template <typename real, typename T, bool BG>
__global__ __launch_bounds__(256) void k_import_state(FPtr<real> D, CPtr<T> src, FPtr<real> B, Layout L, int64_t pitch,
                                                      double gamma, DevScalars *sc) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const real gam = (real)gamma, gm1 = (real)(gamma - 1.0);
    double cx = 0.0, cy = 0.0;
    int bad = 0;
    if (i < L.nx) {
        for (int j = blockIdx.y; j < L.ny; j += gridDim.y) {
            const int64_t e = eidx(L, i, j);
            real u[NF], b[NBG] = {0, 0, 0, 0};
#pragma unroll
            for (int f = 0; f < NF; ++f) u[f] = (real)src.p[f][(int64_t)j * pitch + i];
            if (BG) {
#pragma unroll
                for (int f = 0; f < NBG; ++f) b[f] = B.p[f][e];
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) D.p[f][e] = u[f];
            cell_speeds<real>(u, b[0], b[1], b[2], b[3], gam, gm1, cx, cy, bad);
        }
    }
    block_speeds(cx, cy, bad, sc, 0);
}

// wave speeds of a state without a background into accumulator slot 0
template <typename real>
__global__ __launch_bounds__(256) void k_wavespeed(FPtr<real> U, Layout L, double gamma, DevScalars *sc) {
    const real gam = (real)gamma, gm1 = (real)(gamma - 1.0), zero = (real)0;
    double cx = 0.0, cy = 0.0;
    int bad = 0;
    const int64_t n = (int64_t)L.nx * L.ny;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = eidx(L, (int)(k % L.nx), (int)(k / L.nx));
        real u[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) u[f] = U.p[f][e];
        cell_speeds<real>(u, zero, zero, zero, zero, gam, gm1, cx, cy, bad);
    }
    block_speeds(cx, cy, bad, sc, 0);
}

__global__ void k_reset_scalars(DevScalars *sc, double t0, int *unfilled) {
    *unfilled = 1;
    sc->t = t0;
    sc->dt = 0.0;
    sc->cmax = 0.0;
    sc->t_end = 0.0;
    speed_set(sc->acc[0]);
    speed_set(sc->acc[1]);
    sc->last_cx = sc->last_cy = sc->last_cmax = 0.0;
    sc->steps = 0;
    sc->steps0 = 0;
    sc->cur = 0;
    sc->active = 1;
    sc->nonphys = 0;
    sc->prev_active = 0;
}

// dt for the step about to start (CFL time step with the end-time clamp);
// `prev`: the step before it, of the same call, ends first (one launch for
// both); otherwise the call begins here.  One wave: it runs alone between two
// steps, so its time is that of its chain of loads, and all are issued at once.
__global__ __launch_bounds__(64) void k_step_begin(DevScalars *sc, double t_end, StepConsts k, int prev) {
    const int lane = threadIdx.x;
    const unsigned long long v = speeds_by_lane(sc->acc, lane);
    const int active = sc->active, cur0 = sc->cur, nonphys = sc->nonphys;
    const long long steps = sc->steps;
    const double dt0 = sc->dt, t0 = sc->t;
    const bool end = prev && active;
    const int cur = end ? cur0 ^ 1 : cur0;
    const double cx = __longlong_as_double((long long)__shfl(v, 32 * cur));
    const double cy = __longlong_as_double((long long)__shfl(v, 32 * cur + 1));
    speeds_clear_by_lane(sc->acc[cur ^ 1], lane);
    if (lane) return;
    const double t = end ? t0 + dt0 : t0;
    if (prev) sc->prev_active = active;
    else sc->steps0 = steps;
    if (end) {
        sc->t = t;
        sc->steps = steps + 1;
        sc->cur = cur;
    }
    step_open(sc, t_end, k, t, nonphys, cx, cy);
}

__global__ void k_step_end(DevScalars *sc) { step_end_dev(sc); }

// step start of decomposed stepping: the maxima over every subdomain replace
// this subdomain's own, so that all subdomains take one dt and one c_max.
// From a device array (dc != nullptr) the values are checked here: one that
// is not finite, negative, or zero along a direction with more than one cell
// stops stepping like a non-physical state.
__device__ __forceinline__ void step_begin_global_dev(DevScalars *sc, double cx, double cy, bool check,
                                                      const StepConsts &k) {
    if (check) {
        const bool ok = isfinite(cx) && isfinite(cy) && cx >= 0.0 && cy >= 0.0 && (!k.ax || cx > 0.0) &&
                        (!k.ay || cy > 0.0);
        if (!ok) sc->nonphys = 1;
    }
    speed_set(sc->acc[sc->cur], (unsigned long long)__double_as_longlong(cx), (unsigned long long)__double_as_longlong(cy));
    step_begin_dev(sc, 0.0, k);
}

__global__ void k_step_begin_global(DevScalars *sc, double cx, double cy, const double *dc, StepConsts k) {
    if (dc) {
        cx = dc[0];
        cy = dc[1];
    }
    step_begin_global_dev(sc, cx, cy, dc != nullptr, k);
}

// The step scalars of every subdomain of a domain, by one block of 256
// threads: the step before ends (prev); the maxima over all of them begin the
// next (next).  As separate launches this was one to end each, one to clear
// the maxima, one to raise them and one to begin each.
template <typename real>
__global__ __launch_bounds__(256) void k_domain_scalars(const BatchInst<real> *__restrict__ inst, int n, int prev,
                                                        int next, double *cmax) {
    __shared__ unsigned long long red[2][256];
    unsigned long long m0 = 0ull, m1 = 0ull;
    for (int i = threadIdx.x; i < n; i += 256) {
        DevScalars *sc = inst[i].sc;
        if (prev) step_end_dev(sc);
        const unsigned long long a = speed_max(sc->acc[sc->cur], 0), b = speed_max(sc->acc[sc->cur], 1);
        m0 = a > m0 ? a : m0;
        m1 = b > m1 ? b : m1;
    }
    if (!next) return;
    red[0][threadIdx.x] = m0;
    red[1][threadIdx.x] = m1;
    for (int h = 128; h > 0; h >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < h) {
            for (int d = 0; d < 2; ++d) {
                const unsigned long long o = red[d][threadIdx.x + h];
                if (o > red[d][threadIdx.x]) red[d][threadIdx.x] = o;
            }
        }
    }
    __syncthreads();
    const double cx = __longlong_as_double((long long)red[0][0]), cy = __longlong_as_double((long long)red[1][0]);
    if (threadIdx.x == 0) {
        cmax[0] = cx;
        cmax[1] = cy;
    }
    for (int i = threadIdx.x; i < n; i += 256) step_begin_global_dev(inst[i].sc, cx, cy, true, inst[i].sk);
}

// The ghost cells of every exchange side of every subdomain, each read
// straight from the cell of the neighbour (or the diagonal neighbour) that it
// images; one launch per stage in place of a pack and an unpack per subdomain
// and direction.
template <typename real>
__global__ __launch_bounds__(256) void k_domain_ghosts(const BatchInst<real> *__restrict__ inst, int stage, int px,
                                                       int py) {
    const int sub = blockIdx.z, f = blockIdx.y;
    const BatchInst<real> &I = inst[sub];
    const int nx = I.L.nx, ny = I.L.ny, W = nx + 2 * G, rows = 2 * G * W, n = rows + 2 * G * ny;
    real *S = const_cast<real *>(I.st[stage].S[f]);
    for (int k = blockIdx.x * 256 + threadIdx.x; k < n; k += gridDim.x * 256) {
        int i, j;
        if (k < rows) {
            const int g = k / W;
            i = k % W - G;
            j = g < G ? g - G : ny + g - G;
        } else {
            const int g = (k - rows) % (2 * G);
            j = (k - rows) / (2 * G);
            i = g < G ? g - G : nx + g - G;
        }
        const int ox = i < 0 ? -1 : (i >= nx ? 1 : 0), oy = j < 0 ? -1 : (j >= ny ? 1 : 0);
        if (ox && !(I.exchange & (ox < 0 ? 1 : 2))) continue;   // read through the side's map instead
        if (oy && !(I.exchange & (oy < 0 ? 4 : 8))) continue;
        const int a = (sub % px + ox + px) % px, b = (sub / px + oy + py) % py;
        const BatchInst<real> &N = inst[a + b * px];
        const int si = ox < 0 ? N.L.nx + i : (ox > 0 ? i - nx : i);
        const int sj = oy < 0 ? N.L.ny + j : (oy > 0 ? j - ny : j);
        S[eidx(I.L, i, j)] = N.st[stage].S[f][eidx(N.L, si, sj)];
    }
}

// the device stand-in of an all-reduce(max) over subdomains: this context's
// maxima of the current state into a caller array (non-negative doubles
// order as their bit patterns)
__global__ void k_speeds_max(const DevScalars *sc, unsigned long long *dc) {
    if (threadIdx.x < 2) atomicMax(&dc[threadIdx.x], speed_max(sc->acc[sc->cur], threadIdx.x));
}

// conservation sums: per-block partial sums of rows, then a fixed-order final sum
template <typename real>
__global__ void k_sums_partial(FPtr<real> U, Layout L, double *partials, int npart) {
    __shared__ double red[NF][256];
    double acc[NF] = {0, 0, 0, 0, 0, 0};
    for (int j = blockIdx.x; j < L.ny; j += npart)
        for (int i = threadIdx.x; i < L.nx; i += blockDim.x)
            for (int f = 0; f < NF; ++f) acc[f] += (double)U.p[f][eidx(L, i, j)];
    for (int f = 0; f < NF; ++f) red[f][threadIdx.x] = acc[f];
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int f = 0; f < NF; ++f) red[f][threadIdx.x] += red[f][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int f = 0; f < NF; ++f) partials[(int64_t)blockIdx.x * NF + f] = red[f][0];
}

__global__ void k_sums_final(const double *partials, int npart, double *out, double cell) {
    if (threadIdx.x >= NF) return;
    double s = 0.0;
    for (int b = 0; b < npart; ++b) s += partials[(int64_t)b * NF + threadIdx.x];
    out[threadIdx.x] = s * cell;
}

// ------------------------------------------------------------------ host helpers

// how a context's stored cells are read outside each direction
SideMap x_map(const sacx_ctx *c) { return side_map(c->L.nx, c->bc[0], c->bc[1]); }
SideMap y_map(const sacx_ctx *c) { return side_map(c->L.ny, c->bc[2], c->bc[3]); }
// or where they are stored: the ghost cells themselves
SideMap stored_map(int n) { return side_map(n, SACX_EXCHANGE, SACX_EXCHANGE); }

int prof_event(sacx_ctx *c) {
    if (c->ev_used == (int)c->ev_pool->size()) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return -1;
        c->ev_pool->push_back(e);
    }
    int k = c->ev_used++;
    if (hipEventRecord((*c->ev_pool)[k], c->stream) != hipSuccess) return -1;
    return k;
}

struct ProfScope {
    sacx_ctx *c;
    int cls, start;
    ProfScope(sacx_ctx *c_, int cls_) : c(c_), cls(cls_), start(-1) {
        if (c->prof_on) start = prof_event(c);
    }
    ~ProfScope() {
        if (c->prof_on && start >= 0) {
            int stop = prof_event(c);
            if (stop >= 0) c->ev_marks->push_back({cls, start, stop, 1.0});
        }
    }
};

// a launch group over several contexts: each profiled one takes its share of
// the time, by cells
struct SharedProfScope {
    const std::vector<sacx_ctx *> &ctx;
    int cls;
    bool any = false;
    SharedProfScope(const std::vector<sacx_ctx *> &ctx_, int cls_) : ctx(ctx_), cls(cls_) {
        for (sacx_ctx *c : ctx) {
            if (!c->prof_on) continue;
            c->prof_start = prof_event(c);
            any = true;
        }
    }
    ~SharedProfScope() {
        if (!any) return;
        double all = 0.0;
        for (const sacx_ctx *c : ctx) all += (double)c->L.nx * c->L.ny;
        for (sacx_ctx *c : ctx) {
            if (!c->prof_on || c->prof_start < 0) continue;
            const int stop = prof_event(c);
            if (stop >= 0) c->ev_marks->push_back({cls, c->prof_start, stop, (double)c->L.nx * c->L.ny / all});
        }
    }
};


template <typename real>
FPtr<real> fptr(void *const *p, int nf) {
    FPtr<real> f;
    for (int k = 0; k < NF; ++k) f.p[k] = (real *)(k < nf ? p[k] : p[0]);
    return f;
}

// local boundary fill of one direction (0: x over the interior rows, 1: y over
// the padded width, corners included, so x goes first); exchange sides are
// left as the caller unpacked them
template <typename real>
void fill_dir_t(sacx_ctx *c, void *const *fields, int nf, bool gated, int dir) {
    const Layout &L = c->L;
    const DevScalars *sc = gated ? c->sc : nullptr;
    FPtr<real> S = fptr<real>(fields, nf);
    const int T = 256;
    const int lo = c->bc[2 * dir], hi = c->bc[2 * dir + 1];
    const int n = dir == 0 ? L.nx : L.ny;
    const int along = dir == 0 ? L.ny : L.nx + 2 * G;
    const int skip = (lo == SACX_EXCHANGE ? 1 : 0) | (hi == SACX_EXCHANGE ? 2 : 0);
    if (skip == 3) return;
    if (lo == SACX_PERIODIC && n >= G) {
        // self-exchange: what the low side packed becomes the high halo and vice versa
        void *const *h = dir == 0 ? c->hx : c->hy;
        dim3 g((along + T - 1) / T, nf, 2);
        if (dir == 0) {
            hipLaunchKernelGGL(k_pack_x<real>, g, dim3(T), 0, c->stream, S, nf, L, (real *)h[0], (real *)h[1], 2, sc);
            hipLaunchKernelGGL(k_unpack_x<real>, g, dim3(T), 0, c->stream, S, nf, L, (const real *)h[1],
                               (const real *)h[0], 2, sc);
        } else {
            hipLaunchKernelGGL(k_pack_y<real>, g, dim3(T), 0, c->stream, S, nf, L, stored_map(L.nx), (real *)h[0],
                               (real *)h[1], 2, sc);
            hipLaunchKernelGGL(k_unpack_y<real>, g, dim3(T), 0, c->stream, S, nf, L, (const real *)h[1],
                               (const real *)h[0], 2, sc);
        }
    } else {
        dim3 g((along + T - 1) / T, nf);
        const int periodic = lo == SACX_PERIODIC ? 1 : 0;
        if (dir == 0)
            hipLaunchKernelGGL(k_fill_x<real>, g, dim3(T), 0, c->stream, S, nf, L, periodic, skip, sc);
        else
            hipLaunchKernelGGL(k_fill_y<real>, g, dim3(T), 0, c->stream, S, nf, L, periodic, skip, sc);
    }
}

bool has_exchange(const sacx_ctx *c) {
    for (int s = 0; s < 4; ++s)
        if (c->bc[s] == SACX_EXCHANGE) return true;
    return false;
}

// a periodic direction with fewer than G cells, whose ghosts are filled
// before the stages (one read of its side map reaches one image)
bool narrow(const sacx_ctx *c, int dir) {
    return c->bc[2 * dir] == SACX_PERIODIC && (dir == 0 ? c->L.nx : c->L.ny) < G;
}

// ghosts of one direction of a stage input (or of the background) where that
// direction is narrow; x before y, as in fill_dir_t
int fill_narrow(sacx_ctx *c, void *const *fields, int nf, bool gated, int dir) {
    if (!narrow(c, dir)) return SACX_OK;
    // a tube's one-row stage reads nothing above or below its row
    if (dir == 1 && c->L.ny == 1 && c->L.nx >= 2 && !c->grid.background_on) return SACX_OK;
    if (c->grid.precision == SACX_FP64) fill_dir_t<double>(c, fields, nf, gated, dir);
    else fill_dir_t<float>(c, fields, nf, gated, dir);
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

int fill_narrow(sacx_ctx *c, void *const *fields, int nf, bool gated) {
    const int rc = fill_narrow(c, fields, nf, gated, 0);
    return rc ? rc : fill_narrow(c, fields, nf, gated, 1);
}

// the ghost cells of the state U (the kernels of the learned coefficient and a
// first stage-level call read them); unfilled: only where that is set
int fill_halo(sacx_ctx *c, const int *unfilled = nullptr) {
    const int64_t n = (int64_t)2 * G * (c->L.nx + 2 * G + c->L.ny);
    const dim3 g((unsigned)std::min<int64_t>((n + 255) / 256, 4096), NF);
    const int4 bc = make_int4(c->bc[0], c->bc[1], c->bc[2], c->bc[3]);
    if (c->grid.precision == SACX_FP64)
        hipLaunchKernelGGL(k_fill_ghosts<double>, g, dim3(256), 0, c->stream, fptr<double>(c->U, NF), c->L, bc, unfilled);
    else
        hipLaunchKernelGGL(k_fill_ghosts<float>, g, dim3(256), 0, c->stream, fptr<float>(c->U, NF), c->L, bc, unfilled);
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

// Before a stage-level call: the ghost cells that a loaded state and a
// background have are filled where no such call needed them yet (filled by the
// pass that loads the state, 8000^2 took 0.9 % longer and four subdomains of
// 512^2 2.6 %).  A capture holds the launches too and does not count as done.
int ghosts_ready(sacx_ctx *c) {
    if (!c->ghosts_due && !c->bg_due) return SACX_OK;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    HIPCHK(hipStreamIsCapturing(c->stream, &cap));
    const bool captured = cap != hipStreamCaptureStatusNone;
    if (c->ghosts_due) {
        const int rc = fill_halo(c, c->unfilled);
        if (rc) return rc;
        hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, c->stream, c->unfilled, 0);
        HIPCHK(hipGetLastError());
        c->ghosts_due = captured;
    }
    if (c->bg_due) {
        for (int dir = 0; dir < 2; ++dir) {
            if (c->grid.precision == SACX_FP64) fill_dir_t<double>(c, c->BG, NBG, false, dir);
            else fill_dir_t<float>(c, c->BG, NBG, false, dir);
        }
        HIPCHK(hipGetLastError());
        c->bg_due = captured;
    }
    return SACX_OK;
}

// the state the next stage differences: U between steps, then w1, w2, w3
void *const *stage_input(sacx_ctx *c) {
    switch (c->stage_next) {
        case 1: return c->B1;
        case 2: return c->B2;
        case 3: return c->B1;
        default: return c->U;
    }
}

// grid spacing and the scheme constants derived from it, in the same FP64
// operations as the defining sequence
void set_spacing(sacx_ctx *c, double dx, double dy) {
    c->dx = dx;
    c->dy = dy;
    const sacx_params *params = &c->params;
    SchemeConsts &k = c->kc;
    k.gamma = params->gamma;
    k.gm1 = params->gamma - 1.0;
    k.igm1 = 1.0 / k.gm1;
    k.i12dx = 1.0 / (12.0 * c->dx);
    k.i12dy = 1.0 / (12.0 * c->dy);
    k.idx = 1.0 / c->dx;
    k.idy = 1.0 / c->dy;
    k.i2dx = 1.0 / (2.0 * c->dx);
    k.i2dy = 1.0 / (2.0 * c->dy);
    for (int m = 0; m < 4; ++m) {
        k.kxs[m] = params->cshk[m] * c->dx * c->dx;
        k.kys[m] = params->cshk[m] * c->dy * c->dy;
    }
    k.third = 1.0 / 3.0;
    k.gx = params->g[0];
    k.gy = params->g[1];
    k.grav = params->g[0] != 0.0 || params->g[1] != 0.0;
}

StepConsts step_consts(const sacx_ctx *c) {
    StepConsts sk;
    sk.cfl = c->params.cfl;
    sk.dx = c->dx;
    sk.dy = c->dy;
    for (int m = 0; m < 4; ++m) sk.c2[m] = c->params.c2[m];
    sk.ax = c->grid.nx > 1;
    sk.ay = c->grid.ny > 1;
    return sk;
}

template <typename real>
StageArgs<real> stage_args(sacx_ctx *c, bool stored = false) {
    StageArgs<real> a;
    std::memset(&a, 0, sizeof(a));
    a.L = c->L;
    a.mx = stored ? stored_map(c->L.nx) : x_map(c);
    a.my = stored ? stored_map(c->L.ny) : y_map(c);
    a.ty = c->ty;
    a.nt = c->nt;
    a.split = c->split;
    a.k = c->kc;
    a.hd_cross_on = c->params.hd_cross_on;
    a.sc = c->sc;
    a.fstride = (int64_t)(((const char *)c->U[1] - (const char *)c->U[0]) / (ptrdiff_t)sizeof(real));
    for (int k = 0; k < NBG; ++k) a.BG[k] = (const real *)(c->grid.background_on ? c->BG[k] : nullptr);
    if (c->sur_on) {
        a.Rs = c->sur_r;
        a.rs_pitch = (int)c->sur_pitch;
        a.rs_plane = c->sur_pitch * c->L.ny;
        a.Rk = c->sur_k;
        a.rs_tile = c->sur.tile;
        a.rs_ntx = (c->L.nx + c->sur.tile - 1) / c->sur.tile;
    }
    return a;
}

template <typename real>
RatioArgs<real> ratio_args(sacx_ctx *c) {
    RatioArgs<real> a;
    for (int f = 0; f < NF; ++f) a.S[f] = (const real *)c->U[f];
    a.L = c->L;
    a.gm1 = c->kc.gm1;
    a.igm1 = c->kc.igm1;
    return a;
}

// surrogate refresh at a step start: predict the ratio planes from U (unless
// the caller supplies them) and check them against the plain ratios of U
int sur_refresh(sacx_ctx *c) {
    int rc = fill_halo(c);
    if (rc) return rc;
    const int nx = c->L.nx, ny = c->L.ny;
    InputNorm nm;
    for (int k = 0; k < 12; ++k) nm.v[k] = c->sur.norm[k];
    const bool fp64 = c->grid.precision == SACX_FP64;
    if (c->sur.d_packed) {
        HIPCHK(fp64 ? launch_cnn_inputs<double>(ratio_args<double>(c), nm, c->sur_x, c->stream)
                    : launch_cnn_inputs<float>(ratio_args<float>(c), nm, c->sur_x, c->stream));
        HIPCHK(cnn_forward_dev(c->sur.d_packed, c->sur_x, 1, ny, nx, c->sur_a1, c->sur_a2, c->sur_a1, c->sur_r, 0,
                               c->sur_pitch * ny, c->sur_pitch, c->stream));
    }
    HIPCHK(fp64 ? launch_hd_check<double>(ratio_args<double>(c), c->sur_r, c->sur_pitch, c->sur.bound, c->sur.tile,
                                          c->sur.metric, c->sur_st, c->sur_k, c->stream)
                : launch_hd_check<float>(ratio_args<float>(c), c->sur_r, c->sur_pitch, c->sur.bound, c->sur.tile,
                                         c->sur.metric, c->sur_st, c->sur_k, c->stream));
    const int64_t ntx = (nx + c->sur.tile - 1) / c->sur.tile, nty = (ny + c->sur.tile - 1) / c->sur.tile;
    c->sur_refreshes += 1;
    c->sur_tiles_checked += ntx * nty;
    return SACX_OK;
}

// the stage kernel addresses field f of a buffer as field 0 + f * fstride
template <typename real>
bool fields_uniform(const StageArgs<real> &a) {
    for (int f = 1; f < NF; ++f) {
        const int64_t o = f * a.fstride;
        if (a.S[f] != a.S[0] + o || a.U[f] != a.U[0] + o || a.A[f] != a.A[0] + o || a.out1[f] != a.out1[0] + o ||
            a.out2[f] != a.out2[0] + o)
            return false;
    }
    for (int k = 1; k < NBG; ++k)
        if (a.BG[0] && a.BG[k] != a.BG[0] + k * a.fstride) return false;
    return true;
}

// stored: the cells outside are the ghost cells as they are
template <typename real>
int run_stage(sacx_ctx *c, int stage, void *const *S, void *const *U, void *const *A, void *const *o1,
              void *const *o2, bool stored = false) {
    StageArgs<real> a = stage_args<real>(c, stored);
    for (int f = 0; f < NF; ++f) {
        a.S[f] = (const real *)S[f];
        a.U[f] = (const real *)(U ? U[f] : S[f]);
        a.A[f] = (const real *)(A ? A[f] : S[f]);
        a.out1[f] = (real *)o1[f];
        a.out2[f] = (real *)(o2 ? o2[f] : o1[f]);
    }
    if (!fields_uniform(a)) return fail(SACX_EINVAL, "internal: stage buffers are not laid out at a uniform field stride");
    if (c->box && !a.Rs) {
        HIPCHK(launch_box<real>(stage, c->params.hd_on != 0, c->box, a, c->stream));
        return SACX_OK;
    }
    HIPCHK(launch_stage<real>(stage, c->params.hd_on != 0, c->grid.background_on != 0, a, c->stream));
    return SACX_OK;
}

// one RK4 step of a tube in one launch, from buffer `from` to buffer `to`
template <typename real>
int tube_step(sacx_ctx *c, void *const *from, void *const *to, bool second) {
    TubeArgs<real> a;
    a.U = (const real *)from[0];
    a.out = (real *)to[0];
    a.fstride = (int64_t)(((const char *)c->U[1] - (const char *)c->U[0]) / (ptrdiff_t)sizeof(real));
    for (int f = 1; f < NF; ++f)
        if ((const real *)from[f] != a.U + f * a.fstride || (real *)to[f] != a.out + f * a.fstride)
            return fail(SACX_EINVAL, "internal: state buffers are not laid out at a uniform field stride");
    a.L = c->L;
    a.periodic = c->bc[0] == SACX_PERIODIC;
    a.open_lo = c->bc[0] == SACX_OPEN;
    a.open_hi = c->bc[1] == SACX_OPEN;
    a.k = c->kc;
    a.sc = c->sc;
    a.second = second;
    HIPCHK(launch_tube_step<real>(c->params.hd_on != 0, c->cus, a, c->stream));
    return SACX_OK;
}

// a step without hyper-diffusion in two launches, from `from` to `to`
template <typename real>
int pair_step(sacx_ctx *c, void *const *from, void *const *to, bool second) {
    for (int h = 0; h < 2; ++h) {
        ProfScope ps(c, h ? 3 : 1);
        StageArgs<real> a = stage_args<real>(c);
        for (int f = 0; f < NF; ++f) {
            a.S[f] = (const real *)(h ? c->B2[f] : from[f]);
            a.U[f] = (const real *)from[f];
            a.A[f] = (const real *)c->A[f];
            a.out1[f] = (real *)(h ? to[f] : c->B2[f]);
            a.out2[f] = (real *)c->A[f];
        }
        if (!fields_uniform(a)) return fail(SACX_EINVAL, "internal: stage buffers are not laid out at a uniform field stride");
        HIPCHK(launch_pair<real>(h != 0, second, c->pair_rows, a, c->stream));
    }
    return SACX_OK;
}

int stage(sacx_ctx *c, int s, void *const *S, void *const *U, void *const *A, void *const *o1, void *const *o2) {
    if (narrow(c, 0) || narrow(c, 1)) {
        ProfScope ps(c, 4);
        int rc = fill_narrow(c, S, NF, true);
        if (rc) return rc;
    }
    ProfScope ps(c, s - 1);
    return c->grid.precision == SACX_FP64 ? run_stage<double>(c, s, S, U, A, o1, o2)
                                          : run_stage<float>(c, s, S, U, A, o1, o2);
}

int initial_speeds(sacx_ctx *c) {
    const int64_t n = (int64_t)c->L.nx * c->L.ny;
    const dim3 g((unsigned)std::min<int64_t>((n + 255) / 256, 2048)), t(256);
    if (c->grid.precision == SACX_FP64)
        hipLaunchKernelGGL(k_wavespeed<double>, g, t, 0, c->stream, fptr<double>(c->U, NF), c->L, c->params.gamma, c->sc);
    else
        hipLaunchKernelGGL(k_wavespeed<float>, g, t, 0, c->stream, fptr<float>(c->U, NF), c->L, c->params.gamma, c->sc);
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

template <typename real, typename T>
void import_state(sacx_ctx *c, const void *const *src, int64_t pitch) {
    CPtr<T> t;
    for (int k = 0; k < NF; ++k) t.p[k] = (const T *)src[k];
    // about 8 blocks per compute unit, each over several rows
    const int gx = (c->L.nx + 255) / 256;
    const dim3 g(gx, std::max(1, std::min(c->L.ny, 2048 / gx)));
    if (c->grid.background_on)
        hipLaunchKernelGGL((k_import_state<real, T, true>), g, dim3(256), 0, c->stream, fptr<real>(c->U, NF), t,
                           fptr<real>(c->BG, NBG), c->L, pitch, c->params.gamma, c->sc);
    else
        hipLaunchKernelGGL((k_import_state<real, T, false>), g, dim3(256), 0, c->stream, fptr<real>(c->U, NF), t,
                           fptr<real>(c->U, NF), c->L, pitch, c->params.gamma, c->sc);
}

struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) { ok = false; return; }
        if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
    }
    ~DeviceGuard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

}  // namespace

// ------------------------------------------------------------------ C ABI

extern "C" {

int sacx_abi_version(void) { return SACX_ABI_VERSION; }

const char *sacx_strerror(int code) {
    switch (code) {
        case SACX_OK: return "success";
        case SACX_EINVAL: return "invalid argument";
        case SACX_ENOSPC: return "workspace or buffer too small";
        case SACX_EDEVICE: return "HIP runtime error";
        case SACX_ENONPHYS: return "non-physical state (rho <= 0, p <= 0 or non-finite)";
        case SACX_EUNSUP: return "unsupported request";
        case SACX_ESTATE: return "call out of order";
        default: return "unknown status code";
    }
}

const char *sacx_last_error(void) { return g_last_error.c_str(); }

int sacx_workspace_size(const sacx_grid *grid, const sacx_params *params, size_t *bytes) {
    int rc = check_grid(grid, params);
    if (rc) return rc;
    if (!bytes) return fail(SACX_EINVAL, "bytes must not be NULL");
    *bytes = make_plan(grid).total;
    return SACX_OK;
}

int sacx_create(const sacx_grid *grid, const sacx_params *params, void *d_ws, size_t ws_bytes, void *hip_stream,
                sacx_ctx **out) {
    int rc = check_grid(grid, params);
    if (rc) return rc;
    if (!out) return fail(SACX_EINVAL, "out must not be NULL");
    *out = nullptr;
    if (!d_ws) return fail(SACX_EINVAL, "workspace pointer is NULL");
    if (((uintptr_t)d_ws) % kAlign) return fail(SACX_EINVAL, "workspace must be 256-byte aligned");
    Plan P = make_plan(grid);
    if (ws_bytes < P.total)
        return fail(SACX_ENOSPC, "workspace has %zu bytes, %zu needed", ws_bytes, P.total);
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    sacx_ctx *c = new (std::nothrow) sacx_ctx();
    if (!c) return fail(SACX_EINVAL, "out of host memory");
    std::memset((void *)c, 0, sizeof(*c));
    c->grid = *grid;
    c->params = *params;
    c->device = dev;
    c->stream = (hipStream_t)hip_stream;
    c->L = P.L;
    c->elem = P.elem;
    for (int s = 0; s < 4; ++s) c->bc[s] = SACX_PERIODIC;
    c->ws = (char *)d_ws;
    c->ws_bytes = ws_bytes;
    c->sc = (DevScalars *)(c->ws + P.off_sc);
    c->sums = (double *)(c->ws + P.off_sums);
    c->unfilled = (int *)(c->sums + NF);
    c->partials = (double *)(c->ws + P.off_part);
    c->npart = (int)std::min<int64_t>(kPartials, grid->ny);
    char *st = c->ws + P.off_state;
    for (int f = 0; f < NF; ++f) {
        c->U[f] = st + (0 * NF + f) * P.field_bytes;
        c->B1[f] = st + (1 * NF + f) * P.field_bytes;
        c->B2[f] = st + (2 * NF + f) * P.field_bytes;
        c->A[f] = st + (3 * NF + f) * P.field_bytes;
    }
    for (int k = 0; k < NBG; ++k) c->BG[k] = grid->background_on ? c->ws + P.off_bg + k * P.field_bytes : nullptr;
    c->hx[0] = c->ws + P.off_hx;
    c->hx[1] = c->ws + P.off_hx + P.hx_bytes;
    c->hy[0] = c->ws + P.off_hy;
    c->hy[1] = c->ws + P.off_hy + P.hy_bytes;
    c->split = 1;
    c->nt_auto = c->ty_auto = true;
    set_spacing(c, (grid->x1 - grid->x0) / grid->nx, (grid->y1 - grid->y0) / grid->ny);
    c->initialized = false;
    c->prof_on = false;
    c->sur_on = false;
    c->sur_r = nullptr;
    c->sur_k = nullptr;
    c->ev_pool = new (std::nothrow) std::vector<hipEvent_t>();
    c->ev_marks = new (std::nothrow) std::vector<ProfMark>();
    if (!c->ev_pool || !c->ev_marks) {
        delete c->ev_pool;
        delete c->ev_marks;
        delete c;
        return fail(SACX_EINVAL, "out of host memory");
    }
    c->ev_used = 0;
    auto_rows(c);
    *out = c;
    return SACX_OK;
}

int sacx_destroy(sacx_ctx *ctx) {
    if (!ctx) return SACX_OK;
    {
        // the caller frees the workspace after this call: the work queued
        // on it must be finished first
        DeviceGuard dg(ctx->device);
        (void)hipStreamSynchronize(ctx->stream);
    }
    if (ctx->ev_pool) {
        for (hipEvent_t e : *ctx->ev_pool) (void)hipEventDestroy(e);
        delete ctx->ev_pool;
    }
    delete ctx->ev_marks;
    delete ctx;
    return SACX_OK;
}

int sacx_set_launch(sacx_ctx *ctx, int32_t threads, int32_t rows) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (threads != 0 && threads != 64 && threads != 128 && threads != 256)
        return fail(SACX_EINVAL, "threads must be 64, 128 or 256 (got %d)", threads);
    if (rows < 0 || rows > 4096) return fail(SACX_EINVAL, "rows must be in 1..4096 (got %d)", rows);
    ctx->gen += 1;
    if (threads || rows) ctx->box = 0;
    if (threads) {
        ctx->nt = threads;
        ctx->nt_auto = false;
    } else if (rows && ctx->nt_auto) {
        // rows alone: with the default width, not the one chosen for the automatic height
        ctx->nt = ctx->grid.precision == SACX_FP64 ? 128 : 256;
        ctx->nt_auto = false;
    }
    if (rows) {
        ctx->ty = rows;
        ctx->ty_auto = false;
    } else if (threads && ctx->ty_auto) {
        DeviceGuard dg(ctx->device);
        auto_rows(ctx);
    }
    return SACX_OK;
}

int sacx_set_launch_auto(sacx_ctx *ctx) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    ctx->gen += 1;
    ctx->nt_auto = ctx->ty_auto = true;
    DeviceGuard dg(ctx->device);
    auto_rows(ctx);
    return SACX_OK;
}

int sacx_set_column_split(sacx_ctx *ctx, int32_t on) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (on != 0 && on != 1) return fail(SACX_EINVAL, "on must be 0 or 1 (got %d)", on);
    ctx->split = on;
    ctx->gen += 1;
    if (ctx->ty_auto) {
        DeviceGuard dg(ctx->device);
        auto_rows(ctx);
    }
    return SACX_OK;
}

int sacx_get_launch(const sacx_ctx *ctx, int32_t *threads, int32_t *rows) {
    if (!ctx || !threads || !rows) return fail(SACX_EINVAL, "ctx/threads/rows must not be NULL");
    const bool box = ctx->box && !ctx->sur_on;
    *threads = box ? 64 : ctx->nt;
    *rows = box ? ctx->box : ctx->ty;
    return SACX_OK;
}

int sacx_profile_enable(sacx_ctx *ctx, int32_t on) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    std::memset(&ctx->prof, 0, sizeof(ctx->prof));
    ctx->ev_marks->clear();
    ctx->ev_used = 0;
    ctx->prof_on = on != 0;
    return SACX_OK;
}

int sacx_profile_read(sacx_ctx *ctx, sacx_profile *out) {
    if (!ctx || !out) return fail(SACX_EINVAL, "ctx/out must not be NULL");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    HIPCHK(hipStreamSynchronize(ctx->stream));
    for (const ProfMark &m : *ctx->ev_marks) {
        float whole = 0.f;
        HIPCHK(hipEventElapsedTime(&whole, (*ctx->ev_pool)[m.start], (*ctx->ev_pool)[m.stop]));
        const double ms = whole * m.share;
        if (m.cls < 4) {
            ctx->prof.ms_stage[m.cls] += ms;
            ctx->prof.n_stage[m.cls] += 1;
        } else if (m.cls == 4) {
            ctx->prof.ms_halo += ms;
            ctx->prof.n_halo += 1;
        } else if (m.cls == 6) {
            ctx->prof.ms_surrogate += ms;
            ctx->prof.n_surrogate += 1;
        } else {
            ctx->prof.ms_scalar += ms;
            ctx->prof.n_scalar += 1;
        }
    }
    ctx->ev_marks->clear();
    ctx->ev_used = 0;
    *out = ctx->prof;
    return SACX_OK;
}

int sacx_set_boundaries(sacx_ctx *ctx, const int32_t bc[4]) {
    if (!ctx || !bc) return fail(SACX_EINVAL, "ctx/bc must not be NULL");
    bool exch = false;
    for (int s = 0; s < 4; ++s) {
        if (bc[s] != SACX_PERIODIC && bc[s] != SACX_OPEN && bc[s] != SACX_EXCHANGE)
            return fail(SACX_EINVAL, "bc[%d] = %d is not a boundary kind", s, bc[s]);
        exch = exch || bc[s] == SACX_EXCHANGE;
    }
    if ((bc[0] == SACX_PERIODIC) != (bc[1] == SACX_PERIODIC))
        return fail(SACX_EINVAL, "periodic x boundaries must be paired");
    if ((bc[2] == SACX_PERIODIC) != (bc[3] == SACX_PERIODIC))
        return fail(SACX_EINVAL, "periodic y boundaries must be paired");
    if (ctx->grid.nx == 1 && bc[0] != SACX_PERIODIC) return fail(SACX_EINVAL, "a one-cell direction must be periodic");
    if (ctx->grid.ny == 1 && bc[2] != SACX_PERIODIC) return fail(SACX_EINVAL, "a one-cell direction must be periodic");
    if (ctx->sur_on)
        for (int s = 0; s < 4; ++s)
            if (bc[s] != SACX_PERIODIC)
                return fail(SACX_ESTATE, "the surrogate's ratio planes are periodic: clear it before opening a boundary");
    if (exch && ctx->grid.background_on)
        return fail(SACX_EUNSUP, "exchange boundaries are not supported with a background");
    if ((bc[0] == SACX_EXCHANGE || bc[1] == SACX_EXCHANGE) && ctx->grid.nx < G)
        return fail(SACX_EUNSUP, "an exchange side needs at least %d cells across", G);
    if ((bc[2] == SACX_EXCHANGE || bc[3] == SACX_EXCHANGE) && ctx->grid.ny < G)
        return fail(SACX_EUNSUP, "an exchange side needs at least %d cells across", G);
    for (int s = 0; s < 4; ++s) ctx->bc[s] = bc[s];
    ctx->gen += 1;
    if (ctx->initialized && ctx->grid.background_on) {
        // the static background's ghosts follow the new boundaries
        DeviceGuard dg(ctx->device);
        if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
        ctx->bg_due = true;
        return fill_narrow(ctx, ctx->BG, NBG, false);
    }
    return SACX_OK;
}

// the step scalars of a new state; finish_init fills the narrow ghosts once its fields are in place
static void begin_init(sacx_ctx *ctx, double t0) {
    hipLaunchKernelGGL(k_reset_scalars, dim3(1), dim3(1), 0, ctx->stream, ctx->sc, t0, ctx->unfilled);
}

static int finish_init(sacx_ctx *ctx) {
    HIPCHK(hipGetLastError());
    int rc = fill_narrow(ctx, ctx->U, NF, false);
    if (rc) return rc;
    ctx->stage_next = 0;
    ctx->ghosts_due = true;
    ctx->bg_due = ctx->grid.background_on != 0;
    ctx->initialized = true;
    return SACX_OK;
}

int sacx_init_state(sacx_ctx *ctx, const void *const *d_fields, const void *const *d_bg, int64_t pitch,
                    int32_t in_precision, double t0) {
    if (!ctx || !d_fields) return fail(SACX_EINVAL, "ctx/fields must not be NULL");
    for (int f = 0; f < NF; ++f)
        if (!d_fields[f]) return fail(SACX_EINVAL, "field pointer %d is NULL", f);
    if (pitch < ctx->grid.nx) return fail(SACX_EINVAL, "pitch %lld < nx %d", (long long)pitch, ctx->grid.nx);
    if (in_precision != SACX_FP64 && in_precision != SACX_FP32) return fail(SACX_EINVAL, "bad input precision");
    if (ctx->grid.background_on && !d_bg) return fail(SACX_EINVAL, "background arrays required (background_on)");
    if (ctx->grid.background_on)
        for (int k = 0; k < NBG; ++k)
            if (!d_bg[k]) return fail(SACX_EINVAL, "background pointer %d is NULL", k);
    if (!std::isfinite(t0)) return fail(SACX_EINVAL, "t0 must be finite");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const Layout &L = ctx->L;
    const bool f64 = ctx->grid.precision == SACX_FP64, in64 = in_precision == SACX_FP64;
    begin_init(ctx, t0);
    if (ctx->grid.background_on) {
        const dim3 g((L.nx + 255) / 256, L.ny);
        CPtr<double> bd;
        CPtr<float> bf;
        for (int k = 0; k < NF; ++k) {
            bd.p[k] = (const double *)d_bg[k < NBG ? k : 0];
            bf.p[k] = (const float *)d_bg[k < NBG ? k : 0];
        }
        if (f64 && in64) hipLaunchKernelGGL((k_import<double, double>), g, dim3(256), 0, ctx->stream, fptr<double>(ctx->BG, NBG), bd, NBG, L, pitch);
        else if (f64) hipLaunchKernelGGL((k_import<double, float>), g, dim3(256), 0, ctx->stream, fptr<double>(ctx->BG, NBG), bf, NBG, L, pitch);
        else if (in64) hipLaunchKernelGGL((k_import<float, double>), g, dim3(256), 0, ctx->stream, fptr<float>(ctx->BG, NBG), bd, NBG, L, pitch);
        else hipLaunchKernelGGL((k_import<float, float>), g, dim3(256), 0, ctx->stream, fptr<float>(ctx->BG, NBG), bf, NBG, L, pitch);
        int rc = fill_narrow(ctx, ctx->BG, NBG, false);
        if (rc) return rc;
    }
    if (f64 && in64) import_state<double, double>(ctx, d_fields, pitch);
    else if (f64) import_state<double, float>(ctx, d_fields, pitch);
    else if (in64) import_state<float, double>(ctx, d_fields, pitch);
    else import_state<float, float>(ctx, d_fields, pitch);
    return finish_init(ctx);
}

int sacx_init_problem(sacx_ctx *ctx, int32_t kind, const double *prm, int32_t nprm, double t0) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (kind != SACX_PROBLEM_ORSZAG_TANG && kind != SACX_PROBLEM_BRIO_WU) return fail(SACX_EINVAL, "unknown problem %d", kind);
    const int maxp = kind == SACX_PROBLEM_ORSZAG_TANG ? 1 : 2;
    if (nprm < 0 || nprm > maxp) return fail(SACX_EINVAL, "problem %d takes at most %d parameters", kind, maxp);
    if (nprm > 0 && !prm) return fail(SACX_EINVAL, "prm must not be NULL when nprm > 0");
    if (!std::isfinite(t0)) return fail(SACX_EINVAL, "t0 must be finite");
    if (ctx->grid.background_on) return fail(SACX_EUNSUP, "the problem generators set no background");
    const double p0 = nprm >= 1 ? prm[0] : 1.0, p1 = nprm >= 2 ? prm[1] : 1.0;
    if (!std::isfinite(p0) || !std::isfinite(p1)) return fail(SACX_EINVAL, "parameters must be finite");
    if (kind == SACX_PROBLEM_BRIO_WU && (!(p0 > 0.0) || !(p1 > 0.0)))
        return fail(SACX_EINVAL, "the shock tube's scale factors must be > 0");
    const sacx_grid &g = ctx->grid;
    const int along_y = kind == SACX_PROBLEM_BRIO_WU && g.nx == 1 && g.ny > 1;
    int32_t bc[4] = {SACX_PERIODIC, SACX_PERIODIC, SACX_PERIODIC, SACX_PERIODIC};
    if (kind == SACX_PROBLEM_BRIO_WU) {
        if (along_y) bc[2] = bc[3] = SACX_OPEN;
        else bc[0] = bc[1] = SACX_OPEN;
    }
    int rc = sacx_set_boundaries(ctx, bc);
    if (rc) return rc;
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const double hx = (g.x1 - g.x0) / g.nx, hy = (g.y1 - g.y0) / g.ny;
    const double mid = along_y ? (g.y0 + g.y1) * 0.5 : (g.x0 + g.x1) * 0.5;
    const Layout &L = ctx->L;
    dim3 grd((L.nx + 255) / 256, L.ny);
    if (g.precision == SACX_FP64)
        hipLaunchKernelGGL(k_init_problem<double>, grd, dim3(256), 0, ctx->stream, fptr<double>(ctx->U, NF), L, kind,
                           g.x0, hx, g.y0, hy, mid, along_y, ctx->params.gamma, p0, p1);
    else
        hipLaunchKernelGGL(k_init_problem<float>, grd, dim3(256), 0, ctx->stream, fptr<float>(ctx->U, NF), L, kind,
                           g.x0, hx, g.y0, hy, mid, along_y, ctx->params.gamma, p0, p1);
    begin_init(ctx, t0);
    rc = initial_speeds(ctx);
    return rc ? rc : finish_init(ctx);
}

int sacx_advance(sacx_ctx *ctx, int32_t nsteps, double t_end, int32_t *steps_done, double *t_now) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (nsteps < 0) return fail(SACX_EINVAL, "nsteps must be >= 0");
    if (!std::isfinite(t_end)) return fail(SACX_EINVAL, "t_end must be finite");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    if (has_exchange(ctx)) return fail(SACX_ESTATE, "a context with exchange boundaries steps with sacx_stage");
    if (ctx->stage_next) return fail(SACX_ESTATE, "a step begun with sacx_stage is in progress");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const bool sync = steps_done || t_now;
    const StepConsts sk = step_consts(ctx);
    // a tube's steps take one launch each, but for the last of an odd number
    const bool tube = ctx->L.ny == 1 && ctx->L.nx >= 2 && !ctx->grid.background_on && !ctx->sur_on;
    // and without hyper-diffusion two
    const bool pairs = !tube && stage_pairs(ctx);
    const int whole_steps = tube || pairs ? nsteps & ~1 : 0;
    // A synchronising call enqueues in chunks and stops early once the device
    // reports that stepping ended (end time reached or non-physical state).
    const int chunk = sync ? 128 : (nsteps > 0 ? nsteps : 1);
    for (int n0 = 0; n0 < nsteps; n0 += chunk) {
        const int n1 = std::min(nsteps, n0 + chunk);
        for (int n = n0; n < n1; ++n) {
            {
                ProfScope ps(ctx, 5);
                hipLaunchKernelGGL(k_step_begin, dim3(1), dim3(64), 0, ctx->stream, ctx->sc, t_end, sk, n > 0);
            }
            int rc;
            if (ctx->sur_on) {
                if (ctx->sur_since % ctx->sur.refresh_every == 0) {
                    ProfScope ps(ctx, 6);
                    if ((rc = sur_refresh(ctx))) return rc;
                }
                ctx->sur_since += 1;
            }
            if (n < whole_steps) {
                // in pairs, U to another buffer and back, so that a call ends with its state in U
                const bool second = n & 1;
                if (pairs) {
                    void *const *from = second ? ctx->B1 : ctx->U, *const *to = second ? ctx->U : ctx->B1;
                    if ((rc = ctx->grid.precision == SACX_FP64 ? pair_step<double>(ctx, from, to, second)
                                                               : pair_step<float>(ctx, from, to, second)))
                        return rc;
                    continue;
                }
                ProfScope ps(ctx, 0);
                void *const *from = second ? ctx->B2 : ctx->U, *const *to = second ? ctx->U : ctx->B2;
                if ((rc = ctx->grid.precision == SACX_FP64 ? tube_step<double>(ctx, from, to, second)
                                                           : tube_step<float>(ctx, from, to, second)))
                    return rc;
                continue;
            }
            if ((rc = stage(ctx, 1, ctx->U, nullptr, nullptr, ctx->B1, nullptr))) return rc;
            if ((rc = stage(ctx, 2, ctx->B1, ctx->U, nullptr, ctx->B2, ctx->A))) return rc;
            if ((rc = stage(ctx, 3, ctx->B2, ctx->U, nullptr, ctx->B1, nullptr))) return rc;
            if ((rc = stage(ctx, 4, ctx->B1, nullptr, ctx->A, ctx->U, nullptr))) return rc;
            HIPCHK(hipGetLastError());
        }
        if (sync && n1 < nsteps) {
            int act = 1;
            HIPCHK(hipMemcpyAsync(&act, &ctx->sc->active, sizeof(act), hipMemcpyDeviceToHost, ctx->stream));
            HIPCHK(hipStreamSynchronize(ctx->stream));
            if (!act) break;
        }
    }
    if (nsteps > 0) {
        ProfScope ps(ctx, 5);
        hipLaunchKernelGGL(k_step_end, dim3(1), dim3(1), 0, ctx->stream, ctx->sc);
        HIPCHK(hipGetLastError());
    }
    if (sync) {
        DevScalars h;
        HIPCHK(hipMemcpyAsync(&h, ctx->sc, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
        HIPCHK(hipStreamSynchronize(ctx->stream));
        if (steps_done) *steps_done = nsteps > 0 ? (int32_t)(h.steps - h.steps0) : 0;
        if (t_now) *t_now = h.t;
        if (h.nonphys) return fail(SACX_ENONPHYS, "non-physical state after %lld steps", h.steps);
    }
    return SACX_OK;
}

int sacx_read_fields(sacx_ctx *ctx, void *const *d_out, int64_t pitch, uint32_t field_mask, int32_t out_precision) {
    if (!ctx || !d_out) return fail(SACX_EINVAL, "ctx/out must not be NULL");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    if (pitch < ctx->grid.nx) return fail(SACX_EINVAL, "pitch < nx");
    if (out_precision != SACX_FP64 && out_precision != SACX_FP32) return fail(SACX_EINVAL, "bad output precision");
    if (field_mask & ~0x3Fu) return fail(SACX_EINVAL, "field_mask has bits beyond the 6 fields");
    for (int f = 0; f < NF; ++f)
        if ((field_mask & (1u << f)) && !d_out[f]) return fail(SACX_EINVAL, "output pointer %d is NULL", f);
    if (!field_mask) return SACX_OK;
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    const Layout &L = ctx->L;
    dim3 g((L.nx + 255) / 256, L.ny);
    MPtr<double> td;
    MPtr<float> tf;
    for (int f = 0; f < NF; ++f) {
        void *p = (field_mask & (1u << f)) ? d_out[f] : nullptr;
        td.p[f] = (double *)p;
        tf.p[f] = (float *)p;
    }
    if (ctx->grid.precision == SACX_FP64) {
        if (out_precision == SACX_FP64)
            hipLaunchKernelGGL((k_export<double, double>), g, dim3(256), 0, ctx->stream, fptr<double>(ctx->U, NF), td, field_mask, L, pitch);
        else
            hipLaunchKernelGGL((k_export<double, float>), g, dim3(256), 0, ctx->stream, fptr<double>(ctx->U, NF), tf, field_mask, L, pitch);
    } else {
        if (out_precision == SACX_FP64)
            hipLaunchKernelGGL((k_export<float, double>), g, dim3(256), 0, ctx->stream, fptr<float>(ctx->U, NF), td, field_mask, L, pitch);
        else
            hipLaunchKernelGGL((k_export<float, float>), g, dim3(256), 0, ctx->stream, fptr<float>(ctx->U, NF), tf, field_mask, L, pitch);
    }
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

int sacx_diagnostics(sacx_ctx *ctx, sacx_diag *out) {
    if (!ctx || !out) return fail(SACX_EINVAL, "ctx/out must not be NULL");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    if (ctx->grid.precision == SACX_FP64)
        hipLaunchKernelGGL(k_sums_partial<double>, dim3(ctx->npart), dim3(256), 0, ctx->stream,
                           fptr<double>(ctx->U, NF), ctx->L, ctx->partials, ctx->npart);
    else
        hipLaunchKernelGGL(k_sums_partial<float>, dim3(ctx->npart), dim3(256), 0, ctx->stream,
                           fptr<float>(ctx->U, NF), ctx->L, ctx->partials, ctx->npart);
    hipLaunchKernelGGL(k_sums_final, dim3(1), dim3(64), 0, ctx->stream, (const double *)ctx->partials, ctx->npart,
                       ctx->sums, ctx->dx * ctx->dy);
    HIPCHK(hipGetLastError());
    DevScalars h;
    double sums[NF];
    HIPCHK(hipMemcpyAsync(&h, ctx->sc, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(hipMemcpyAsync(sums, ctx->sums, sizeof(sums), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    const double cx = __builtin_bit_cast(double, speed_max(h.acc[h.cur], 0));
    const double cy = __builtin_bit_cast(double, speed_max(h.acc[h.cur], 1));
    out->t = h.t;
    out->dt = h.dt;
    out->c_x = cx;
    out->c_y = cy;
    const int ax = ctx->grid.nx > 1, ay = ctx->grid.ny > 1;
    out->c_max = (ax && ay) ? std::max(cx, cy) : (ax ? cx : cy);
    for (int f = 0; f < NF; ++f) out->sums[f] = sums[f];
    out->steps = h.steps;
    out->nonphys = h.nonphys;
    return SACX_OK;
}

int sacx_halo_buffer_size(const sacx_ctx *ctx, int32_t side, size_t *bytes) {
    if (!ctx || !bytes) return fail(SACX_EINVAL, "ctx/bytes must not be NULL");
    if (side < 0 || side > 3) return fail(SACX_EINVAL, "side must be 0..3");
    const size_t along = side < 2 ? (size_t)ctx->grid.ny : (size_t)ctx->grid.nx + 2 * G;
    *bytes = (size_t)NF * G * along * ctx->elem;
    return SACX_OK;
}

// stored: the corners of a packed y strip are the ghost cells as they are;
// otherwise the cells that the x sides' boundary has there
static int halo_io(sacx_ctx *ctx, int32_t side, void *buf, bool pack, bool stored) {
    if (!ctx || !buf) return fail(SACX_EINVAL, "ctx/buffer must not be NULL");
    if (side < 0 || side > 3) return fail(SACX_EINVAL, "side must be 0..3");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    const Layout &L = ctx->L;
    if ((side < 2 && L.nx < G) || (side >= 2 && L.ny < G))
        return fail(SACX_EUNSUP, "halo exchange needs at least %d cells across", G);
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    if (stored) {
        const int rc = ghosts_ready(ctx);
        if (rc) return rc;
    }
    const SideMap mx = stored ? stored_map(L.nx) : x_map(ctx);
    ProfScope ps(ctx, 4);
    const int T = 256;
    const int s = side & 1;
    const bool f64 = ctx->grid.precision == SACX_FP64;
    void *const *S = stage_input(ctx);
    if (side < 2) {
        dim3 g((L.ny + T - 1) / T, NF, 1);
        if (f64) {
            if (pack) hipLaunchKernelGGL(k_pack_x<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, (double *)buf, (double *)buf, 10 + s, (const DevScalars *)nullptr);
            else hipLaunchKernelGGL(k_unpack_x<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, (const double *)buf, (const double *)buf, 10 + s, (const DevScalars *)nullptr);
        } else {
            if (pack) hipLaunchKernelGGL(k_pack_x<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, (float *)buf, (float *)buf, 10 + s, (const DevScalars *)nullptr);
            else hipLaunchKernelGGL(k_unpack_x<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, (const float *)buf, (const float *)buf, 10 + s, (const DevScalars *)nullptr);
        }
    } else {
        dim3 g((L.nx + 2 * G + T - 1) / T, NF, 1);
        if (f64) {
            if (pack) hipLaunchKernelGGL(k_pack_y<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, mx, (double *)buf, (double *)buf, 10 + s, (const DevScalars *)nullptr);
            else hipLaunchKernelGGL(k_unpack_y<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, (const double *)buf, (const double *)buf, 10 + s, (const DevScalars *)nullptr);
        } else {
            if (pack) hipLaunchKernelGGL(k_pack_y<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, mx, (float *)buf, (float *)buf, 10 + s, (const DevScalars *)nullptr);
            else hipLaunchKernelGGL(k_unpack_y<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, (const float *)buf, (const float *)buf, 10 + s, (const DevScalars *)nullptr);
        }
    }
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

int sacx_halo_pack(sacx_ctx *ctx, int32_t side, void *d_buf) { return halo_io(ctx, side, d_buf, true, true); }

int sacx_halo_unpack(sacx_ctx *ctx, int32_t side, const void *d_buf) {
    return halo_io(ctx, side, const_cast<void *>(d_buf), false, true);
}

// ------------------------------------------------------------------ decomposed stepping

int sacx_fill_boundaries(sacx_ctx *ctx, int32_t direction) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (direction != 0 && direction != 1) return fail(SACX_EINVAL, "direction must be 0 (x) or 1 (y)");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    ProfScope ps(ctx, 4);
    if (ctx->grid.precision == SACX_FP64) fill_dir_t<double>(ctx, stage_input(ctx), NF, false, direction);
    else fill_dir_t<float>(ctx, stage_input(ctx), NF, false, direction);
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

// stored: the stage reads the ghost cells as they are; otherwise the sides' maps
static int stage_call(sacx_ctx *ctx, const double *c_max, int32_t c_max_on_device, int32_t *stage_done, bool stored) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (c_max_on_device != 0 && c_max_on_device != 1) return fail(SACX_EINVAL, "c_max_on_device must be 0 or 1");
    if (c_max_on_device && !c_max) return fail(SACX_EINVAL, "a device c_max must not be NULL");
    if (c_max_on_device && ((uintptr_t)c_max % alignof(double)))
        return fail(SACX_EINVAL, "a device c_max must be 8-byte aligned");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    if (ctx->sur_on) return fail(SACX_ESTATE, "a context with a learned coefficient steps with sacx_advance");
    if (ctx->stage_next == 0 && c_max && !c_max_on_device) {
        for (int d = 0; d < 2; ++d)
            if (!std::isfinite(c_max[d]) || c_max[d] < 0.0) return fail(SACX_EINVAL, "c_max[%d] must be finite and >= 0", d);
        if ((ctx->grid.nx > 1 && !(c_max[0] > 0.0)) || (ctx->grid.ny > 1 && !(c_max[1] > 0.0)))
            return fail(SACX_EINVAL, "c_max must be > 0 along every direction with more than one cell");
    }
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    int rc;
    if (stored && (rc = ghosts_ready(ctx))) return rc;
    const int s = ctx->stage_next + 1;
    if (s == 1) {
        ProfScope ps(ctx, 5);
        if (c_max_on_device)
            hipLaunchKernelGGL(k_step_begin_global, dim3(1), dim3(1), 0, ctx->stream, ctx->sc, 0.0, 0.0, c_max,
                               step_consts(ctx));
        else if (c_max)
            hipLaunchKernelGGL(k_step_begin_global, dim3(1), dim3(1), 0, ctx->stream, ctx->sc, c_max[0], c_max[1],
                               (const double *)nullptr, step_consts(ctx));
        else
            hipLaunchKernelGGL(k_step_begin, dim3(1), dim3(64), 0, ctx->stream, ctx->sc, 0.0, step_consts(ctx), 0);
        HIPCHK(hipGetLastError());
    }
    {
        ProfScope ps(ctx, s - 1);
        void *const *S[4] = {ctx->U, ctx->B1, ctx->B2, ctx->B1};
        void *const *O1[4] = {ctx->B1, ctx->B2, ctx->B1, ctx->U};
        void *const *U = s == 2 || s == 3 ? ctx->U : nullptr, *const *A = s == 4 ? ctx->A : nullptr;
        void *const *O2 = s == 2 ? ctx->A : nullptr;
        rc = ctx->grid.precision == SACX_FP64 ? run_stage<double>(ctx, s, S[s - 1], U, A, O1[s - 1], O2, stored)
                                              : run_stage<float>(ctx, s, S[s - 1], U, A, O1[s - 1], O2, stored);
    }
    if (rc) return rc;
    if (s == 4) {
        ProfScope ps(ctx, 5);
        hipLaunchKernelGGL(k_step_end, dim3(1), dim3(1), 0, ctx->stream, ctx->sc);
        HIPCHK(hipGetLastError());
    }
    ctx->stage_next = s & 3;
    if (stage_done) *stage_done = s;
    return SACX_OK;
}

int sacx_stage(sacx_ctx *ctx, const double *c_max, int32_t c_max_on_device, int32_t *stage_done) {
    return stage_call(ctx, c_max, c_max_on_device, stage_done, true);
}

int sacx_set_spacing(sacx_ctx *ctx, double dx, double dy) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    if (!std::isfinite(dx) || !std::isfinite(dy) || !(dx > 0.0) || !(dy > 0.0))
        return fail(SACX_EINVAL, "dx and dy must be finite and > 0");
    if (ctx->stage_next) return fail(SACX_ESTATE, "a step begun with sacx_stage is in progress");
    set_spacing(ctx, dx, dy);
    ctx->gen += 1;
    return SACX_OK;
}

int sacx_wave_speeds_max(sacx_ctx *ctx, double *d_c_max) {
    if (!ctx || !d_c_max) return fail(SACX_EINVAL, "ctx/d_c_max must not be NULL");
    if ((uintptr_t)d_c_max % alignof(double)) return fail(SACX_EINVAL, "d_c_max must be 8-byte aligned");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    if (ctx->stage_next) return fail(SACX_ESTATE, "a step begun with sacx_stage is in progress");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    hipLaunchKernelGGL(k_speeds_max, dim3(1), dim3(64), 0, ctx->stream, (const DevScalars *)ctx->sc,
                       (unsigned long long *)d_c_max);
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

int sacx_wave_speeds(sacx_ctx *ctx, double c_max[2]) {
    if (!ctx || !c_max) return fail(SACX_EINVAL, "ctx/c_max must not be NULL");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    DevScalars h;
    HIPCHK(hipMemcpyAsync(&h, ctx->sc, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    c_max[0] = __builtin_bit_cast(double, speed_max(h.acc[h.cur], 0));
    c_max[1] = __builtin_bit_cast(double, speed_max(h.acc[h.cur], 1));
    return SACX_OK;
}

// ------------------------------------------------------------------ surrogate

}  // extern "C"

namespace {

__global__ void k_fill_f32(float *p, int64_t n, float v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_zero_stats(HdDevStats *st) {
    unsigned long long *p = (unsigned long long *)st;
    const int n = (int)(sizeof(HdDevStats) / sizeof(unsigned long long));
    for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) p[i] = 0ull;
}

struct SurPlan {
    int64_t pitch;
    size_t off_r, off_st, off_k, off_x, off_a1, off_a2, total;
};

SurPlan sur_plan(const sacx_ctx *c) {
    SurPlan p;
    const int64_t nx = c->L.nx, ny = c->L.ny;
    p.pitch = (int64_t)round_up((size_t)nx, 64);
    size_t o = 0;
    p.off_r = o;  o = round_up(o + (size_t)10 * p.pitch * ny * sizeof(float), kAlign);
    p.off_st = o; o = round_up(o + sizeof(HdDevStats), kAlign);
    // one flag per check tile, sized for the smallest tile (one cell)
    p.off_k = o;  o = round_up(o + (size_t)nx * ny, kAlign);
    p.off_x = o;  o = round_up(o + (size_t)nx * ny * 8 * 2, kAlign);
    p.off_a1 = o; o = round_up(o + (size_t)nx * ny * 32 * 2, kAlign);
    p.off_a2 = o; o = round_up(o + (size_t)nx * ny * 32 * 2, kAlign);
    p.total = o;
    return p;
}

int sur_supported(const sacx_ctx *c) {
    if (!c->params.hd_on) return fail(SACX_EUNSUP, "the surrogate replaces hyper-diffusion ratios: hd_on must be 1");
    if (c->grid.background_on) return fail(SACX_EUNSUP, "the surrogate needs a context without background");
    for (int s = 0; s < 4; ++s)
        if (c->bc[s] != SACX_PERIODIC) return fail(SACX_EUNSUP, "the surrogate needs periodic boundaries on every side");
    if (c->L.ny < 2) return fail(SACX_EUNSUP, "the surrogate needs ny >= 2");
    if (c->L.nx % 32 != 0) return fail(SACX_EUNSUP, "the surrogate needs nx to be a multiple of 32 (got %d)", c->L.nx);
    return SACX_OK;
}

}  // namespace

extern "C" {

int sacx_surrogate_workspace_size(const sacx_ctx *ctx, size_t *bytes) {
    if (!ctx || !bytes) return fail(SACX_EINVAL, "ctx/bytes must not be NULL");
    *bytes = sur_plan(ctx).total;
    return SACX_OK;
}

int sacx_hd_set_surrogate(sacx_ctx *ctx, const sacx_surrogate *cfg, void *d_ws, size_t ws_bytes) {
    if (!ctx || !cfg || !d_ws) return fail(SACX_EINVAL, "ctx/cfg/workspace must not be NULL");
    int rc = sur_supported(ctx);
    if (rc) return rc;
    if (cfg->refresh_every < 1) return fail(SACX_EINVAL, "refresh_every must be >= 1");
    if (cfg->tile < 1) return fail(SACX_EINVAL, "tile must be >= 1");
    if (cfg->metric != SACX_HD_CHECK_RATIO && cfg->metric != SACX_HD_CHECK_FLUX)
        return fail(SACX_EINVAL, "metric must be SACX_HD_CHECK_RATIO or SACX_HD_CHECK_FLUX");
    if (!(cfg->bound >= 0.0)) return fail(SACX_EINVAL, "bound must be >= 0");
    for (int k = 0; k < 12; ++k)
        if (!std::isfinite(cfg->norm[k])) return fail(SACX_EINVAL, "input normalisation must be finite");
    if ((uintptr_t)d_ws % kAlign) return fail(SACX_EINVAL, "surrogate workspace must be 256-byte aligned");
    if (cfg->d_packed && (uintptr_t)cfg->d_packed % 16) return fail(SACX_EINVAL, "packed weights must be 16-byte aligned");
    const SurPlan p = sur_plan(ctx);
    if (ws_bytes < p.total)
        return fail(SACX_ENOSPC, "surrogate workspace too small (%zu < %zu bytes)", ws_bytes, p.total);
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    char *w = (char *)d_ws;
    ctx->sur = *cfg;
    ctx->sur_pitch = p.pitch;
    ctx->sur_r = (float *)(w + p.off_r);
    ctx->sur_st = (HdDevStats *)(w + p.off_st);
    ctx->sur_k = (unsigned char *)(w + p.off_k);
    ctx->sur_x = w + p.off_x;
    ctx->sur_a1 = w + p.off_a1;
    ctx->sur_a2 = w + p.off_a2;
    ctx->sur_since = 0;
    ctx->sur_refreshes = 0;
    ctx->sur_tiles_checked = 0;
    const int64_t nr = (int64_t)10 * p.pitch * ctx->L.ny;
    hipLaunchKernelGGL(k_fill_f32, dim3(1024), dim3(256), 0, ctx->stream, ctx->sur_r, nr, -1.0f);
    // every tile flag 0 (fallen back) until the first check (its bytes as
    // float zeros: the flag region is a whole number of 256-byte blocks)
    const int64_t nk = (int64_t)(p.off_x - p.off_k) / 4;
    hipLaunchKernelGGL(k_fill_f32, dim3(256), dim3(256), 0, ctx->stream, (float *)ctx->sur_k, nk, 0.0f);
    hipLaunchKernelGGL(k_zero_stats, dim3(1), dim3(64), 0, ctx->stream, ctx->sur_st);
    HIPCHK(hipGetLastError());
    ctx->sur_on = true;
    return SACX_OK;
}

int sacx_hd_clear_surrogate(sacx_ctx *ctx) {
    if (!ctx) return fail(SACX_EINVAL, "ctx must not be NULL");
    ctx->sur_on = false;
    ctx->sur_r = nullptr;
    ctx->sur_k = nullptr;
    return SACX_OK;
}

int sacx_hd_ratio_buffer(sacx_ctx *ctx, float **d_r, int64_t *pitch) {
    if (!ctx || !d_r || !pitch) return fail(SACX_EINVAL, "ctx/d_r/pitch must not be NULL");
    if (!ctx->sur_on) return fail(SACX_ESTATE, "the surrogate is not set");
    *d_r = ctx->sur_r;
    *pitch = ctx->sur_pitch;
    return SACX_OK;
}

int sacx_hd_read_stats(sacx_ctx *ctx, sacx_hd_stats *out) {
    if (!ctx || !out) return fail(SACX_EINVAL, "ctx/out must not be NULL");
    if (!ctx->sur_on) return fail(SACX_ESTATE, "the surrogate is not set");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    HdDevStats h;
    HIPCHK(hipMemcpyAsync(&h, ctx->sur_st, sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    out->refreshes = ctx->sur_refreshes;
    out->tiles_checked = ctx->sur_tiles_checked;
    // reduce the counters' copies (maxima of non-negative doubles are the
    // maxima of their bit patterns)
    unsigned long long nf = 0, bu = 0, ba = 0;
    for (int k = 0; k < kStatSlots; ++k) {
        nf += h.tiles_fallback[k];
        bu = std::max(bu, h.err_used[k]);
        ba = std::max(ba, h.err_all[k]);
    }
    out->tiles_fallback = (int64_t)nf;
    double eu, ea;
    std::memcpy(&eu, &bu, sizeof(eu));
    std::memcpy(&ea, &ba, sizeof(ea));
    out->err_used = eu;
    out->err_all = ea;
    return SACX_OK;
}

int sacx_cnn_inputs(sacx_ctx *ctx, const float norm[12], void *d_x) {
    if (!ctx || !norm || !d_x) return fail(SACX_EINVAL, "ctx/norm/x must not be NULL");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    if (ctx->grid.background_on) return fail(SACX_EUNSUP, "network inputs need a context without background");
    if ((uintptr_t)d_x % 16) return fail(SACX_EINVAL, "input buffer must be 16-byte aligned");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    InputNorm nm;
    for (int k = 0; k < 12; ++k) nm.v[k] = norm[k];
    HIPCHK(ctx->grid.precision == SACX_FP64 ? launch_cnn_inputs<double>(ratio_args<double>(ctx), nm, d_x, ctx->stream)
                                            : launch_cnn_inputs<float>(ratio_args<float>(ctx), nm, d_x, ctx->stream));
    return SACX_OK;
}

int sacx_hd_ratio_fields(sacx_ctx *ctx, float *d_r, float *d_d1, int64_t pitch) {
    if (!ctx || !d_r) return fail(SACX_EINVAL, "ctx/d_r must not be NULL");
    if (!ctx->initialized) return fail(SACX_ESTATE, "sacx_init_state has not been called");
    if (ctx->grid.background_on) return fail(SACX_EUNSUP, "ratio fields need a context without background");
    if (pitch < ctx->L.nx) return fail(SACX_EINVAL, "pitch must be >= nx");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the context device");
    int rc = fill_halo(ctx);
    if (rc) return rc;
    HIPCHK(ctx->grid.precision == SACX_FP64
               ? launch_ratio_fields<double>(ratio_args<double>(ctx), d_r, d_d1, pitch, ctx->stream)
               : launch_ratio_fields<float>(ratio_args<float>(ctx), d_r, d_d1, pitch, ctx->stream));
    return SACX_OK;
}


}  // extern "C"

// ------------------------------------------------------------------ batches

struct sacx_batch {
    int n;
    int precision;
    int device;
    hipStream_t stream;
    std::vector<sacx_ctx *> *ctx;
    char *tab;          // BatchInst array
    int *sync;          // abort flag, queue counters, per-instance completion counters
    BatchItem *items;
    int *qinst;         // instances of each XCD queue; of stage launches, those with narrow y
    int nnarrow, narrow_nx;   // how many those are, and their most columns
    int qoff[kBatchQueues], qlen[kBatchQueues], ioff[kBatchQueues + 1];
    int items_cap;
    int nitems;
    int nt;
    std::vector<int> *rows;
    int box;            // rows of the stage launches' boxes; 0: marching tiles
    bool shape_auto;    // threads and rows chosen by batch_shape (until set explicitly)
    bool stages;        // the tables are those of the stage launches; else of the persistent launch
    bool dirty;
    unsigned long long gen_built;  // sum of the instance generations the table was built from
    int blocks;
};

namespace {

constexpr size_t kInstBytes = sizeof(BatchInst<double>) > sizeof(BatchInst<float>) ? sizeof(BatchInst<double>)
                                                                                    : sizeof(BatchInst<float>);

// ghost-fill pieces of one stage of a batched instance (a tube, one row
// with one-row tiles, fills only the ghost cells of its row)
int batch_fill_pieces(const sacx_grid &g) {
    const bool oned = g.ny == 1 && g.nx >= 2;
    const int64_t cells = (int64_t)NF * ((oned ? 0 : 2LL * G * (g.nx + 2 * G)) + 2LL * G * g.ny);
    return (int)((cells + kBatchFillPiece - 1) / kBatchFillPiece);
}

// entries of one stage's work lists (tiles of at most 58 columns, the
// narrowest tile, and one row; fill pieces)
int64_t batch_items_bound(int n, const sacx_grid *g) {
    int64_t t = 0;
    for (int i = 0; i < n; ++i) {
        const int64_t xt = (g[i].nx + 57) / 58;
        t += (g[i].ny == 1 ? xt : xt * g[i].ny) + batch_fill_pieces(g[i]);
    }
    return t;
}

struct BatchPlan {
    size_t off_tab, off_sync, off_items, off_qinst, off_inst, total;
    std::vector<size_t> inst_off, inst_bytes;
};

int batch_plan(int n, const sacx_grid *grids, const sacx_params *params, BatchPlan *P) {
    if (n < 1 || n > 65536) return fail(SACX_EINVAL, "batch size must be 1..65536");
    if (!grids || !params) return fail(SACX_EINVAL, "grids/params must not be NULL");
    P->inst_off.resize(n);
    P->inst_bytes.resize(n);
    for (int i = 0; i < n; ++i) {
        int rc = check_grid(&grids[i], &params[i]);
        if (rc) return rc;
        if (grids[i].precision != grids[0].precision) return fail(SACX_EINVAL, "all batch instances need one precision");
        if (grids[i].background_on) return fail(SACX_EUNSUP, "batched instances have no background");
        if (grids[i].nx < G) return fail(SACX_EUNSUP, "batched instances need nx >= %d", G);
        if (!params[i].hd_on) return fail(SACX_EUNSUP, "batched instances run with hyper-diffusion on");
        P->inst_bytes[i] = make_plan(&grids[i]).total;
    }
    size_t off = 0;
    P->off_tab = off; off += round_up((size_t)n * kInstBytes, kAlign);
    P->off_sync = off; off += round_up((size_t)(BATCH_SYNC0 + 2 * n) * sizeof(int), kAlign);
    P->off_items = off; off += round_up((size_t)batch_items_bound(n, grids) * sizeof(BatchItem), kAlign);
    P->off_qinst = off; off += round_up((size_t)n * sizeof(int), kAlign);
    P->off_inst = off;
    for (int i = 0; i < n; ++i) { P->inst_off[i] = off; off += round_up(P->inst_bytes[i], kAlign); }
    P->total = off;
    return SACX_OK;
}

// the ghost rows of a stage's input of batched instances whose periodic y has
// fewer than G rows (one launch for all of them: as one per instance, 41 of them
// made 169 launches a step)
template <typename real>
__global__ __launch_bounds__(256) void k_batch_narrow(const BatchInst<real> *__restrict__ inst,
                                                      const int *__restrict__ which, int stage) {
    const BatchInst<real> &I = inst[which[blockIdx.x]];
    if (!I.sc->active) return;
    const Layout L = I.L;
    real *S = const_cast<real *>(I.st[stage].S[blockIdx.y]);
    for (int i = blockIdx.z * 256 + threadIdx.x; i < L.nx; i += gridDim.z * 256)
        for (int g = 1; g <= G; ++g) {
            S[eidx(L, i, -g)] = S[eidx(L, i, (G * L.ny - g) % L.ny)];
            S[eidx(L, i, L.ny - 1 + g)] = S[eidx(L, i, (g - 1) % L.ny)];
        }
}

__global__ void k_zero_ints(int *p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// which kernel runs the stage launches of several contexts with one scheme
template <typename real>
bool many_split(const sacx_ctx *c) {
    // (a tube's one-row tile is the one-thread kernel's)
    return sizeof(real) == 8 && c->params.hd_on && c->split && c->L.ny > 1;
}

template <typename real>
hipError_t many_blocks_per_cu(int cols, bool hd, bool split, int *per) {
    return split ? split_blocks_per_cu_fp64(cols, false, per) : batch_stage_blocks_per_cu<real>(cols, hd, per);
}

constexpr int kTubeCells = 512 - 2 * G;   // a tube's cells per block of the box kernel

// the tiles of one context in a list: boxes of 58 x `box` cells, or (box 0)
// strips of nt columns and `rows` rows
void list_tiles(const sacx_ctx *c, int i, int nt, int rows, int box, std::vector<BatchItem> *out) {
    const bool tube = c->L.ny == 1;
    const int tx = box ? (tube ? kTubeCells : 58) : nt - 2 * G;
    const int ty = tube ? 1 : (box ? box : rows);
    for (int y = 0; y < (c->L.ny + ty - 1) / ty; ++y)
        for (int x = 0; x < (c->L.nx + tx - 1) / tx; ++x) out->push_back({i, x, y, BATCH_TILE});
}

// Columns and strip rows of stage launches over several contexts, as
// shape_for_slots chooses them for one grid: the cheapest (time per row) x
// (rows + 9) over the widths and the numbers of blocks per compute unit, the
// rows those that bring the tiles of all the contexts to that many blocks.
// False where none of at most 256 rows fits one round of resident blocks.
template <typename real>
bool shape_for_many(const std::vector<sacx_ctx *> &ctx, int cus, bool split, int *nt, int *rows, int *box) {
    const bool hd = ctx[0]->params.hd_on != 0;
    const int kind = sizeof(real) == 8 ? (hd ? KIND_SPLIT : KIND_F64_NOHD) : (hd ? KIND_F32 : KIND_F32_NOHD);
    double best = 0.0;
    *rows = 256;
    *nt = sizeof(real) == 8 ? 128 : 256;
    auto tiles = [&](int cols, int ty) {
        const int TX = cols - 2 * G;
        int64_t t = 0;
        for (const sacx_ctx *c : ctx)
            if (c->L.ny > 1) t += (int64_t)((c->L.nx + TX - 1) / TX) * ((c->L.ny + ty - 1) / ty);
        return t;
    };
    // the cheapest shape of one round with at most `limit` rows
    auto one_round = [&](int limit) {
        for (int w = 0; w < 3; ++w) {
            const int cols = 64 << w;
            int per = 0;
            if (many_blocks_per_cu<real>(cols, hd, split, &per) != hipSuccess) { (void)hipGetLastError(); continue; }
            for (int k = 1; k <= std::min(per, 8); ++k) {
                const float us = kRowUs[kind][w][k - 1];
                if (us == 0.0f) break;
                int lo = 1, hi = limit + 1;   // the fewest rows whose tiles fit (limit + 1: none)
                while (lo < hi) {
                    const int mid = (lo + hi) / 2;
                    if (tiles(cols, mid) <= (int64_t)cus * k) hi = mid; else lo = mid + 1;
                }
                if (lo > limit) continue;
                const double cost = us * (lo + 9.0);
                if (best == 0.0 || cost < best) { best = cost; *nt = cols; *rows = lo; }
            }
        }
        return best > 0.0;
    };
    if (!one_round(256)) {
        // Strips of up to 512 rows in one round, against several rounds of
        // 256: FP64 only where those are more than 1.3 rounds (two blocks per
        // compute unit).  ms per step: FP64 4 x 2500^2 6.42 -> 5.23, 8 x 2000^2
        // 8.97 -> 6.70, but 4 x 2000^2 (1.06 rounds) 3.39 -> 3.49; FP32 4 x 3000^2
        // (1.13 rounds) 4.77 -> 3.35.
        if (sizeof(real) == 4 || (double)tiles(*nt, 256) > 1.3 * 2.0 * cus) one_round(512);
        *box = 0;
        return false;
    }
    // boxes instead where they are expected to be faster
    int64_t t8 = 0, t16 = 0;
    for (const sacx_ctx *c : ctx) {
        t8 += c->L.ny > 1 ? box_tiles(c->L, 8) : (c->L.nx + kTubeCells - 1) / kTubeCells;
        t16 += c->L.ny > 1 ? box_tiles(c->L, 16) : (c->L.nx + kTubeCells - 1) / kTubeCells;
    }
    bool boxes = false;   // (tubes alone run in blocks of their own width)
    for (const sacx_ctx *c : ctx) boxes = boxes || c->L.ny > 1;
    *box = !boxes ? 0 : box_for(sizeof(real) == 4, hd, t8, t16, cus, best);
    return true;
}

// one context's entry of an instance table, for tiles of nt columns and `rows` rows
template <typename real>
int table_entry(sacx_ctx *c, int nt, int rows, BatchInst<real> *out) {
    BatchInst<real> &I = *out;
    std::memset((void *)&I, 0, sizeof(I));
    void *const *S[4] = {c->U, c->B1, c->B2, c->B1};
    void *const *U[4] = {c->U, c->U, c->U, c->U};
    void *const *A[4] = {c->A, c->A, c->A, c->A};
    void *const *O1[4] = {c->B1, c->B2, c->B1, c->U};
    void *const *O2[4] = {c->B1, c->A, c->B1, c->U};
    for (int st = 0; st < 4; ++st) {
        StageArgs<real> a = stage_args<real>(c);
        a.nt = nt;
        a.ty = rows;
        for (int f = 0; f < NF; ++f) {
            a.S[f] = (const real *)S[st][f];
            a.U[f] = (const real *)U[st][f];
            a.A[f] = (const real *)A[st][f];
            a.out1[f] = (real *)O1[st][f];
            a.out2[f] = (real *)O2[st][f];
        }
        if (!fields_uniform(a)) return fail(SACX_EINVAL, "internal: a context's buffers are not laid out at a uniform field stride");
        I.st[st] = a;
    }
    I.sk = step_consts(c);
    I.sc = c->sc;
    I.L = c->L;
    I.periodic_x = c->bc[0] == SACX_PERIODIC;
    I.periodic_y = c->bc[2] == SACX_PERIODIC;
    I.oned = (c->grid.ny == 1 && c->grid.nx >= 2) ? 1 : 0;
    for (int k = 0; k < 4; ++k) I.exchange |= c->bc[k] == SACX_EXCHANGE ? 1 << k : 0;
    return SACX_OK;
}

// the work lists of the persistent launch: per XCD queue its instances, most
// expensive first, each its fill pieces then its tiles
template <typename real>
void queue_tiles(sacx_batch *b, std::vector<BatchInst<real>> *tab, std::vector<BatchItem> *flat, std::vector<int> *qinst) {
    const int n = b->n, TX = b->nt - 2 * G;
    struct Costed { int64_t cost; BatchItem it; };
    std::vector<std::vector<Costed>> tiles(n);
    std::vector<int64_t> icost(n, 0);
    for (int i = 0; i < n; ++i) {
        const sacx_ctx *c = (*b->ctx)[i];
        BatchInst<real> &I = (*tab)[i];
        const int xt = (c->L.nx + TX - 1) / TX;
        if (I.oned) {
            for (int x = 0; x < xt; ++x) tiles[i].push_back({1, {i, x, 0, BATCH_TILE}});
        } else {
            const int ty = (*b->rows)[i];
            const int yt = (c->L.ny + ty - 1) / ty;
            for (int y = 0; y < yt; ++y) {
                const int rows = std::min(ty, c->L.ny - y * ty);
                for (int x = 0; x < xt; ++x) tiles[i].push_back({(int64_t)rows + 2 * G, {i, x, y, BATCH_TILE}});
            }
        }
        std::stable_sort(tiles[i].begin(), tiles[i].end(), [](const Costed &p, const Costed &q) { return p.cost > q.cost; });
        I.ntiles = (int)tiles[i].size();
        I.nfill = batch_fill_pieces(c->grid);
        for (const Costed &t : tiles[i]) icost[i] += t.cost;
    }
    // instances to the queues, most expensive first to the least loaded
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int p, int q) { return icost[p] > icost[q]; });
    std::vector<std::vector<int>> group(kBatchQueues);
    std::vector<int64_t> load(kBatchQueues, 0);
    for (int i : order) {
        const int k = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        group[k].push_back(i);
        load[k] += icost[i];
    }
    for (int k = 0; k < kBatchQueues; ++k) {
        b->qoff[k] = (int)flat->size();
        b->ioff[k] = (int)qinst->size();
        for (int i : group[k]) {
            qinst->push_back(i);
            for (int p = 0; p < (*tab)[i].nfill; ++p) flat->push_back({i, p, 0, BATCH_FILL});
            for (const Costed &t : tiles[i]) flat->push_back(t.it);
        }
        b->qlen[k] = (int)flat->size() - b->qoff[k];
    }
    b->ioff[kBatchQueues] = (int)qinst->size();
}

template <typename real>
int batch_build(sacx_batch *b) {
    const int n = b->n;
    int cus = 0;
    HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device));
    b->box = 0;
    if (b->shape_auto && b->stages) {
        int rows = 0;
        shape_for_many<real>(*b->ctx, cus, false, &b->nt, &rows, &b->box);
        for (int i = 0; i < n; ++i) {
            const int ny = (*b->ctx)[i]->grid.ny;
            (*b->rows)[i] = ny == 1 ? 1 : std::min(rows, ny);
        }
    }
    std::vector<BatchInst<real>> tab(n);
    for (int i = 0; i < n; ++i) {
        int rc = table_entry<real>((*b->ctx)[i], b->nt, (*b->rows)[i], &tab[i]);
        if (rc) return rc;
    }
    std::vector<BatchItem> flat;
    std::vector<int> qinst;
    if (b->stages) {
        // the boxes' tiles, instance by instance, then the tubes'
        for (int tube = 0; tube < 2; ++tube)
            for (int i = 0; i < n; ++i)
                if (tab[i].oned == tube) list_tiles((*b->ctx)[i], i, b->nt, (*b->rows)[i], b->box, &flat);
        b->narrow_nx = 0;
        for (int i = 0; i < n; ++i) {
            const sacx_ctx *c = (*b->ctx)[i];
            if (tab[i].oned || !narrow(c, 1)) continue;
            qinst.push_back(i);
            b->narrow_nx = std::max(b->narrow_nx, c->L.nx);
        }
        b->nnarrow = (int)qinst.size();
        qinst.resize(n, 0);
    } else {
        queue_tiles(b, &tab, &flat, &qinst);
        int per_cu = 0;
        HIPCHK(batch_blocks_per_cu<real>(b->nt, &per_cu));
        if (per_cu < 1) return fail(SACX_EUNSUP, "batched kernel does not fit on a compute unit with %d threads", b->nt);
        b->blocks = per_cu * cus;
    }
    if ((int64_t)flat.size() > b->items_cap) return fail(SACX_ENOSPC, "batch work list exceeds its bound");
    b->nitems = (int)flat.size();
    HIPCHK(hipMemcpyAsync(b->qinst, qinst.data(), sizeof(int) * n, hipMemcpyHostToDevice, b->stream));
    HIPCHK(hipMemcpyAsync(b->tab, tab.data(), sizeof(BatchInst<real>) * n, hipMemcpyHostToDevice, b->stream));
    HIPCHK(hipMemcpyAsync(b->items, flat.data(), sizeof(BatchItem) * flat.size(), hipMemcpyHostToDevice, b->stream));
    // host vectors go out of scope: finish the copies first
    HIPCHK(hipStreamSynchronize(b->stream));
    b->dirty = false;
    return SACX_OK;
}

template <typename real>
void batch_args(const sacx_batch *b, int nsteps, int spin, BatchArgs<real> *a) {
    a->inst = (const BatchInst<real> *)b->tab;
    a->n = b->n;
    a->items = b->items;
    a->qinst = b->qinst;
    for (int k = 0; k < kBatchQueues; ++k) { a->qoff[k] = b->qoff[k]; a->qlen[k] = b->qlen[k]; a->ioff[k] = b->ioff[k]; }
    a->ioff[kBatchQueues] = b->ioff[kBatchQueues];
    a->sync = b->sync;
    a->nsteps = nsteps;
    a->spin_limit = spin;
}

// nsteps steps by stage launches; the word behind the abort flag collects the
// instances' non-physical flags after the last one
template <typename real>
int batch_stages(sacx_batch *b, int nsteps) {
    BatchArgs<real> a;
    batch_args(b, 0, 0, &a);
    int *flag = b->sync + BATCH_QUEUE0;
    hipLaunchKernelGGL(k_zero_ints, dim3(1), dim3(64), 0, b->stream, flag, 1);
    for (int s = 0; s < nsteps; ++s) {
        HIPCHK(launch_batch_scalars<real>(a, s > 0, true, flag, b->stream));
        for (int st = 1; st <= 4; ++st) {
            // (x has at least G cells)
            if (b->nnarrow)
                hipLaunchKernelGGL(k_batch_narrow<real>, dim3(b->nnarrow, NF, std::min((b->narrow_nx + 255) / 256, 64)),
                                   dim3(256), 0, b->stream, a.inst, (const int *)b->qinst, st - 1);
            HIPCHK(b->box ? launch_batch_box<real>(a, b->box, st, true, b->nitems, b->stream)
                          : launch_batch_stage<real>(a, b->nt, st, true, b->nitems, b->stream));
        }
    }
    HIPCHK(launch_batch_scalars<real>(a, nsteps > 0, false, flag, b->stream));
    return SACX_OK;
}

}  // namespace

extern "C" {

int sacx_batch_workspace_size(int32_t n, const sacx_grid *grids, const sacx_params *params, size_t *bytes) {
    if (!bytes) return fail(SACX_EINVAL, "bytes must not be NULL");
    BatchPlan P;
    int rc = allocating([&] { return batch_plan(n, grids, params, &P); });
    if (rc) return rc;
    *bytes = P.total;
    return SACX_OK;
}

int sacx_batch_destroy(sacx_batch *b) {
    if (!b) return SACX_OK;
    {
        DeviceGuard dg(b->device);
        (void)hipStreamSynchronize(b->stream);
    }
    if (b->ctx)
        for (sacx_ctx *c : *b->ctx) sacx_destroy(c);
    delete b->ctx;
    delete b->rows;
    delete b;
    return SACX_OK;
}

int sacx_batch_create(int32_t n, const sacx_grid *grids, const sacx_params *params, const int32_t *bc, void *d_ws,
                      size_t ws_bytes, void *hip_stream, sacx_batch **out) {
    if (!out) return fail(SACX_EINVAL, "out must not be NULL");
    *out = nullptr;
    BatchPlan P;
    int rc = allocating([&] { return batch_plan(n, grids, params, &P); });
    if (rc) return rc;
    if (!d_ws || ((uintptr_t)d_ws) % kAlign) return fail(SACX_EINVAL, "workspace must be non-NULL and 256-byte aligned");
    if (ws_bytes < P.total) return fail(SACX_ENOSPC, "workspace has %zu bytes, %zu needed", ws_bytes, P.total);
    sacx_batch *b = new (std::nothrow) sacx_batch;
    if (!b) return fail(SACX_EINVAL, "out of host memory");
    std::memset((void *)b, 0, sizeof(*b));
    b->ctx = new (std::nothrow) std::vector<sacx_ctx *>();
    b->rows = new (std::nothrow) std::vector<int>();
    if (!b->ctx || !b->rows) { sacx_batch_destroy(b); return fail(SACX_EINVAL, "out of host memory"); }
    rc = allocating([&] { b->ctx->reserve(n); b->rows->assign(n, 0); return SACX_OK; });
    if (rc) { sacx_batch_destroy(b); return rc; }
    b->n = n;
    b->precision = grids[0].precision;
    b->stream = (hipStream_t)hip_stream;
    if (hipGetDevice(&b->device) != hipSuccess) { sacx_batch_destroy(b); return fail(SACX_EDEVICE, "no current device"); }
    char *ws = (char *)d_ws;
    b->tab = ws + P.off_tab;
    b->sync = (int *)(ws + P.off_sync);
    b->items = (BatchItem *)(ws + P.off_items);
    b->qinst = (int *)(ws + P.off_qinst);
    b->items_cap = (int)batch_items_bound(n, grids);
    hipLaunchKernelGGL(k_zero_ints, dim3(8), dim3(256), 0, b->stream, b->sync, BATCH_SYNC0 + 2 * n);
    if (hipGetLastError() != hipSuccess) {
        sacx_batch_destroy(b);
        return fail(SACX_EDEVICE, "clearing the batch's synchronisation words failed");
    }
    for (int i = 0; i < n; ++i) {
        sacx_ctx *c = nullptr;
        rc = sacx_create(&grids[i], &params[i], ws + P.inst_off[i], P.inst_bytes[i], hip_stream, &c);
        if (rc) { sacx_batch_destroy(b); return rc; }
        b->ctx->push_back(c);
        if (bc) {
            for (int k = 0; k < 4; ++k)
                if (bc[4 * i + k] == SACX_EXCHANGE) {
                    sacx_batch_destroy(b);
                    return fail(SACX_EUNSUP, "instance %d: a batched instance cannot have exchange boundaries", i);
                }
            rc = sacx_set_boundaries(c, bc + 4 * i);
            if (rc) { sacx_batch_destroy(b); return rc; }
        }
    }
    sacx_batch_set_tiles_auto(b);
    *out = b;
    return SACX_OK;
}

int sacx_batch_context(sacx_batch *b, int32_t i, sacx_ctx **out) {
    if (!b || !out) return fail(SACX_EINVAL, "batch/out must not be NULL");
    if (i < 0 || i >= b->n) return fail(SACX_EINVAL, "instance %d out of range", i);
    *out = (*b->ctx)[i];
    return SACX_OK;
}

// the shapes of the persistent launch; the stage launches choose theirs when
// their tables are built
int sacx_batch_set_tiles_auto(sacx_batch *b) {
    if (!b) return fail(SACX_EINVAL, "batch must not be NULL");
    b->nt = b->precision == SACX_FP64 ? 128 : 256;
    for (int i = 0; i < b->n; ++i) {
        const int ny = (*b->ctx)[i]->grid.ny;
        (*b->rows)[i] = ny == 1 ? 1 : std::min(64, ny);
    }
    b->shape_auto = true;
    b->dirty = true;
    return SACX_OK;
}

int sacx_batch_set_tiles(sacx_batch *b, int32_t threads, const int32_t *rows) {
    if (!b) return fail(SACX_EINVAL, "batch must not be NULL");
    if (threads != 0 && threads != 64 && threads != 128 && threads != 256)
        return fail(SACX_EINVAL, "threads must be 64, 128 or 256");
    if (rows)
        for (int i = 0; i < b->n; ++i)
            if (rows[i] < 1 || rows[i] > 4096) return fail(SACX_EINVAL, "rows[%d] = %d out of 1..4096", i, rows[i]);
    if (threads || rows) b->shape_auto = false;
    if (threads) b->nt = threads;
    if (rows)
        for (int i = 0; i < b->n; ++i) (*b->rows)[i] = (*b->ctx)[i]->grid.ny == 1 ? 1 : rows[i];
    b->dirty = true;
    return SACX_OK;
}

int sacx_batch_advance(sacx_batch *b, int32_t nsteps, int32_t sync) {
    if (!b) return fail(SACX_EINVAL, "batch must not be NULL");
    if (nsteps < 0) return fail(SACX_EINVAL, "nsteps must be >= 0");
    unsigned long long gsum = 0;
    for (sacx_ctx *c : *b->ctx) {
        if (!c->initialized) return fail(SACX_ESTATE, "every batch instance needs sacx_init_state first");
        if (has_exchange(c)) return fail(SACX_ESTATE, "a batched instance cannot have exchange boundaries");
        if (c->stage_next) return fail(SACX_ESTATE, "a batched instance has a step begun with sacx_stage in progress");
        if (c->sur_on) return fail(SACX_EUNSUP, "a batched instance has a learned coefficient set: the batch uses the plain one");
        gsum += c->gen;
    }
    DeviceGuard dg(b->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the batch device");
    // One launch per stage over the tiles of every instance, against the
    // persistent launch in which each instance stays on one XCD (us per step):
    // 64 instances of the benchmark's ranges 1018 against 1588, 8 tubes and 8
    // boxes 219 against 925, 3 small tubes and boxes 93 against 274 at its
    // best shape, 12 tubes 24 against 81: a stage launch has no fill entries,
    // no waits between entries and uses the whole chip for every instance.
    // The persistent launch runs where the bound of its waits is set.
    const char *env = getenv("SACX_BATCH_SPIN_LIMIT");
    const bool stages = env == nullptr;
    if (b->dirty || gsum != b->gen_built || stages != b->stages) {
        b->stages = stages;
        b->dirty = true;   // until the tables are complete
        int rc = allocating([&] { return b->precision == SACX_FP64 ? batch_build<double>(b) : batch_build<float>(b); });
        if (rc) return rc;
        b->gen_built = gsum;
    }
    if (b->stages) {
        const int rc = b->precision == SACX_FP64 ? batch_stages<double>(b, nsteps) : batch_stages<float>(b, nsteps);
        if (rc) return rc;
        if (sync) {
            int w[2] = {0, 0};   // the abort flag, and the word behind it
            HIPCHK(hipMemcpyAsync(w, b->sync + BATCH_ABORT, sizeof(w), hipMemcpyDeviceToHost, b->stream));
            HIPCHK(hipStreamSynchronize(b->stream));
            if (w[0]) return fail(SACX_EDEVICE, "a batch dependency wait exceeded its bound; the instance states are undefined");
            if (w[1]) return fail(SACX_ENONPHYS, "a batch instance reached a non-physical state");
        }
        return SACX_OK;
    }
    const int spin = std::max(0, atoi(env));
    // steps per launch: every queue index stays within an int
    int qmax = 1;
    for (int k = 0; k < kBatchQueues; ++k) qmax = std::max(qmax, b->qlen[k]);
    const int per_launch = (int)std::max<int64_t>(1, std::min<int64_t>(4096, (INT32_MAX - 2LL * b->n) / (4LL * qmax)));
    for (int done = 0; done < nsteps; done += per_launch) {
        const int k = std::min(per_launch, nsteps - done);
        // the queue counters, block counts and completion counters start at
        // zero; the abort flag is sticky (a launch after an abandoned one
        // does nothing)
        hipLaunchKernelGGL(k_zero_ints, dim3(8), dim3(256), 0, b->stream, b->sync + BATCH_QUEUE0,
                           BATCH_SYNC0 - BATCH_QUEUE0 + 2 * b->n);
        if (b->precision == SACX_FP64) {
            BatchArgs<double> a;
            batch_args(b, k, spin, &a);
            HIPCHK(launch_batch<double>(a, b->nt, b->blocks, b->stream));
        } else {
            BatchArgs<float> a;
            batch_args(b, k, spin, &a);
            HIPCHK(launch_batch<float>(a, b->nt, b->blocks, b->stream));
        }
    }
    if (sync) {
        // a wait that exceeded its bound left the batch part-way through a
        // launch: report it (the instance states are then undefined, and the
        // flag stays set, so later launches of this batch do nothing)
        int ab = 0;
        HIPCHK(hipMemcpyAsync(&ab, b->sync + BATCH_ABORT, sizeof(int), hipMemcpyDeviceToHost, b->stream));
        HIPCHK(hipStreamSynchronize(b->stream));
        if (ab) return fail(SACX_EDEVICE, "a batch dependency wait exceeded its bound; the instance states are undefined");
    }
    if (sync) {
        HIPCHK(hipStreamSynchronize(b->stream));
        for (sacx_ctx *c : *b->ctx) {
            int np = 0;
            HIPCHK(hipMemcpy(&np, &c->sc->nonphys, sizeof(int), hipMemcpyDeviceToHost));
            if (np) return fail(SACX_ENONPHYS, "a batch instance reached a non-physical state");
        }
    }
    return SACX_OK;
}

}  // extern "C"

// ------------------------------------------------------------------ decomposed domain

namespace {

__global__ void k_zero_doubles(double *p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0.0;
}

constexpr size_t kDomainAlign = 256;

// the neighbour across `side` of subdomain (a, b) in a px x py layout,
// wrapping around the domain (a periodic image is a neighbour too)
int domain_neighbour(int px, int py, int a, int b, int side) {
    switch (side) {
        case 0: return ((a - 1 + px) % px) + b * px;
        case 1: return ((a + 1) % px) + b * px;
        case 2: return a + ((b - 1 + py) % py) * px;
        default: return a + ((b + 1) % py) * px;
    }
}

bool domain_edge(int px, int py, int a, int b, int side) {
    switch (side) {
        case 0: return a == 0;
        case 1: return a == px - 1;
        case 2: return b == 0;
        default: return b == py - 1;
    }
}

}  // namespace

struct sacx_domain {
    int px, py;
    std::vector<sacx_ctx *> *subs;            // row-major, px x py
    std::vector<std::array<void *, 4>> *buf;  // per subdomain and side: the strip it packs (exchange sides)
    std::vector<std::array<int, 4>> *nbr;     // per subdomain and side: the neighbour (exchange sides)
    std::vector<std::array<int, 4>> *bc;      // per subdomain: the boundary kinds the layout was checked with
    double *cmax;                             // the whole domain's wave-speed maxima (device)
    // stage launches over all subdomains: device tables in the caller's
    // buffer and the launch shape
    char *tab;
    BatchItem *items;
    int ntiles, nt, box;
    bool mixed;  // some subdomain's y neighbour has x sides of other kinds
    bool each;   // stage launches by subdomain, in each one's own launch shape
    bool split;
    bool built;
    unsigned long long gen_built;
};

namespace {

size_t domain_tab_bytes(int n) { return round_up((size_t)n * kInstBytes, kDomainAlign); }

// entries of one stage's tile list (tiles of at most 58 columns and one row)
size_t domain_items_bytes(int n, sacx_ctx *const *subs) {
    int64_t t = 0;
    for (int i = 0; i < n; ++i) t += (int64_t)((subs[i]->grid.nx + 57) / 58) * subs[i]->grid.ny;
    return round_up((size_t)t * sizeof(BatchItem), kDomainAlign);
}

// the tables of the stage launches, from the subdomains' current settings
template <typename real>
int domain_build(sacx_domain *d, unsigned long long gen) {
    const std::vector<sacx_ctx *> &subs = *d->subs;
    const int n = (int)subs.size();
    sacx_ctx *c0 = subs[0];
    d->split = true;
    bool set = false;   // a launch shape set on some subdomain
    for (const sacx_ctx *c : subs) {
        d->split = d->split && many_split<real>(c);
        set = set || !c->nt_auto || !c->ty_auto;
    }
    int rows = 0, cus = 0;
    bool one_round = false;
    d->box = 0;
    HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c0->device));
    if (set) d->nt = c0->nt;
    else one_round = shape_for_many<real>(subs, cus, d->split, &d->nt, &rows, &d->box);
    std::vector<BatchInst<real>> tab(n);
    std::vector<BatchItem> items;
    for (const sacx_ctx *c : subs)   // the one-thread tile was asked for
        if (sizeof(real) == 8 && c->params.hd_on && !c->split) d->box = 0;
    for (int i = 0; i < n; ++i) {
        sacx_ctx *c = subs[i];
        const int ty = set ? c->ty : std::min(rows, c->L.ny);
        int rc = table_entry<real>(c, d->nt, ty, &tab[i]);
        if (rc) return rc;
        list_tiles(c, i, d->nt, ty, d->box, &items);
    }
    d->ntiles = (int)items.size();
    // A list of several rounds of blocks against launches by subdomain, each in
    // the shape of its own grid, ms per step: FP64 2000^2 cells each 3.14 and
    // 3.13, 2500^2 5.65 and 4.75, 4000^2 12.5 and 12.0, 2000 x 4000 13.4 and
    // 12.4, but 1000 x 2000 3.16 and 3.31; FP32 4000^2 5.54 and 5.34, 2000 x
    // 4000 5.60 and 5.53, but 2000^2 1.43 and 1.49.
    int64_t cells = INT64_MAX;
    for (const sacx_ctx *c : subs) cells = std::min(cells, (int64_t)c->L.nx * c->L.ny);
    d->each = d->box == 0 && !one_round && cells >= (sizeof(real) == 8 ? 4000000 : 8000000);
    HIPCHK(hipMemcpyAsync(d->tab, tab.data(), sizeof(tab[0]) * n, hipMemcpyHostToDevice, c0->stream));
    HIPCHK(hipMemcpyAsync(d->items, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice, c0->stream));
    // the host vectors go out of scope: finish the copies first
    HIPCHK(hipStreamSynchronize(c0->stream));
    d->gen_built = gen;
    d->built = true;
    return SACX_OK;
}

// nsteps steps, every launch over all subdomains (but the stages of large ones)
template <typename real>
int domain_steps(sacx_domain *d, int nsteps) {
    sacx_ctx *c0 = (*d->subs)[0];
    const int n = d->px * d->py;
    BatchArgs<real> a;
    std::memset((void *)&a, 0, sizeof(a));
    a.inst = (const BatchInst<real> *)d->tab;
    a.n = n;
    a.items = d->items;
    int64_t ghosts = 0;
    bool exchange = false;
    for (const sacx_ctx *c : *d->subs) {
        ghosts = std::max<int64_t>(ghosts, 2 * G * ((int64_t)c->L.nx + 2 * G + c->L.ny));
        exchange = exchange || has_exchange(c);
    }
    const dim3 gg((unsigned)std::min<int64_t>((ghosts + 255) / 256, 1024), NF, n);
    for (int s = 0; s <= nsteps; ++s) {
        {
            SharedProfScope ps(*d->subs, 5);
            hipLaunchKernelGGL(k_domain_scalars<real>, dim3(1), dim3(256), 0, c0->stream, a.inst, n, s > 0, s < nsteps,
                               d->cmax);
        }
        for (int st = 1; st <= 4 && s < nsteps; ++st) {
            if (exchange) {
                SharedProfScope ps(*d->subs, 4);
                hipLaunchKernelGGL(k_domain_ghosts<real>, gg, dim3(256), 0, c0->stream, a.inst, st - 1, d->px, d->py);
            }
            if (d->each) {
                for (sacx_ctx *c : *d->subs) {
                    void *const *S[4] = {c->U, c->B1, c->B2, c->B1};
                    void *const *O[4] = {c->B1, c->B2, c->B1, c->U};
                    const int rc = stage(c, st, S[st - 1], c->U, c->A, O[st - 1], c->A);
                    if (rc) return rc;
                }
                continue;
            }
            SharedProfScope ps(*d->subs, st - 1);
            const int tiles = d->ntiles;
            if (d->box) {
                HIPCHK(launch_batch_box<real>(a, d->box, st, c0->params.hd_on != 0, tiles, c0->stream));
                continue;
            }
            if constexpr (sizeof(real) == 8) {
                if (d->split) {
                    HIPCHK(launch_batch_split_fp64(a, d->nt, st, tiles, c0->stream));
                    continue;
                }
            }
            HIPCHK(launch_batch_stage<real>(a, d->nt, st, c0->params.hd_on != 0, tiles, c0->stream));
        }
    }
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

}  // namespace

extern "C" {

// checks shared by the size query and creation; on success *bytes is the
// caller memory the domain needs
static int domain_check(int32_t px, int32_t py, sacx_ctx *const *subs, size_t *bytes) {
    if (px < 1 || py < 1 || (int64_t)px * py > 4096) return fail(SACX_EINVAL, "px, py must be >= 1 (at most 4096 subdomains)");
    if (!subs || !bytes) return fail(SACX_EINVAL, "subs/bytes must not be NULL");
    const int n = px * py;
    for (int i = 0; i < n; ++i) {
        if (!subs[i]) return fail(SACX_EINVAL, "subdomain %d is NULL", i);
        for (int j = 0; j < i; ++j)
            if (subs[j] == subs[i]) return fail(SACX_EINVAL, "subdomain %d appears twice", i);
    }
    const sacx_ctx *c0 = subs[0];
    size_t total = kDomainAlign;  // the maxima
    for (int b = 0; b < py; ++b)
        for (int a = 0; a < px; ++a) {
            const int i = a + b * px;
            const sacx_ctx *c = subs[i];
            if (!c->initialized) return fail(SACX_ESTATE, "subdomain %d has no state (sacx_init_state)", i);
            if (c->device != c0->device || c->stream != c0->stream)
                return fail(SACX_EINVAL, "subdomain %d is not on the device and stream of subdomain 0", i);
            if (c->grid.precision != c0->grid.precision) return fail(SACX_EINVAL, "subdomain %d has another precision", i);
            if (std::memcmp(&c->params, &c0->params, sizeof(sacx_params)) != 0)
                return fail(SACX_EINVAL, "subdomain %d has other scheme parameters", i);
            if (c->dx != c0->dx || c->dy != c0->dy)
                return fail(SACX_EINVAL, "subdomain %d has another grid spacing (sacx_set_spacing)", i);
            if (c->sur_on) return fail(SACX_ESTATE, "subdomain %d has a learned coefficient", i);
            for (int side = 0; side < 4; ++side) {
                const bool edge = domain_edge(px, py, a, b, side);
                if (c->bc[side] != SACX_EXCHANGE) {
                    if (!edge) return fail(SACX_EINVAL, "subdomain %d side %d borders a subdomain but is not EXCHANGE", i, side);
                    continue;
                }
                const sacx_ctx *nb = subs[domain_neighbour(px, py, a, b, side)];
                if (nb->bc[side ^ 1] != SACX_EXCHANGE)
                    return fail(SACX_EINVAL, "subdomain %d side %d: the neighbour's facing side is not EXCHANGE", i, side);
                if ((side < 2 && nb->grid.ny != c->grid.ny) || (side >= 2 && nb->grid.nx != c->grid.nx))
                    return fail(SACX_EINVAL, "subdomain %d side %d: the neighbour's strip has another length", i, side);
                size_t sb = 0;
                int rc = sacx_halo_buffer_size(c, side, &sb);
                if (rc) return rc;
                total += round_up(sb, kDomainAlign);
            }
        }
    *bytes = total + domain_tab_bytes(n) + domain_items_bytes(n, subs);
    return SACX_OK;
}

int sacx_domain_buffer_size(int32_t px, int32_t py, sacx_ctx *const *subs, size_t *bytes) {
    return domain_check(px, py, subs, bytes);
}

int sacx_domain_create(int32_t px, int32_t py, sacx_ctx *const *subs, void *d_buf, size_t buf_bytes, sacx_domain **out) {
    if (!out) return fail(SACX_EINVAL, "out must not be NULL");
    *out = nullptr;
    size_t need = 0;
    int rc = domain_check(px, py, subs, &need);
    if (rc) return rc;
    if (!d_buf) return fail(SACX_EINVAL, "buffer pointer is NULL");
    if (((uintptr_t)d_buf) % kDomainAlign) return fail(SACX_EINVAL, "buffer must be 256-byte aligned");
    if (buf_bytes < need) return fail(SACX_ENOSPC, "buffer has %zu bytes, %zu needed", buf_bytes, need);
    sacx_domain *d = new (std::nothrow) sacx_domain();
    if (!d) return fail(SACX_EINVAL, "out of host memory");
    d->px = px;
    d->py = py;
    d->built = false;
    rc = allocating([&] {
        d->subs = new std::vector<sacx_ctx *>(subs, subs + (size_t)px * py);
        d->buf = new std::vector<std::array<void *, 4>>((size_t)px * py);
        d->nbr = new std::vector<std::array<int, 4>>((size_t)px * py);
        d->bc = new std::vector<std::array<int, 4>>((size_t)px * py);
        return SACX_OK;
    });
    if (rc) {
        sacx_domain_destroy(d);
        return rc;
    }
    char *p = (char *)d_buf;
    d->cmax = (double *)p;
    p += kDomainAlign;
    d->tab = p;
    p += domain_tab_bytes(px * py);
    d->items = (BatchItem *)p;
    p += domain_items_bytes(px * py, subs);
    for (int b = 0; b < py; ++b)
        for (int a = 0; a < px; ++a) {
            const int i = a + b * px;
            for (int side = 0; side < 4; ++side) {
                (*d->buf)[i][side] = nullptr;
                (*d->nbr)[i][side] = -1;
                (*d->bc)[i][side] = subs[i]->bc[side];
                if (subs[i]->bc[side] != SACX_EXCHANGE) continue;
                size_t sb = 0;
                sacx_halo_buffer_size(subs[i], side, &sb);
                (*d->buf)[i][side] = p;
                const int nb = domain_neighbour(px, py, a, b, side);
                (*d->nbr)[i][side] = nb;
                if (side >= 2 && (subs[nb]->bc[0] != subs[i]->bc[0] || subs[nb]->bc[1] != subs[i]->bc[1])) d->mixed = true;
                p += round_up(sb, kDomainAlign);
            }
        }
    *out = d;
    return SACX_OK;
}

int sacx_domain_destroy(sacx_domain *d) {
    if (!d) return SACX_OK;
    delete d->subs;
    delete d->buf;
    delete d->nbr;
    delete d->bc;
    delete d;
    return SACX_OK;
}

// both strips of one direction of a context's stage input in one launch
// (the two-sided form of the pack / unpack kernels): b0 for the low side,
// b1 for the high side
static int halo_io_both(sacx_ctx *ctx, int dir, void *b0, void *b1, bool pack, bool stored) {
    const SideMap mx = stored ? stored_map(ctx->L.nx) : x_map(ctx);
    ProfScope ps(ctx, 4);
    const Layout &L = ctx->L;
    const int T = 256;
    void *const *S = stage_input(ctx);
    const bool f64 = ctx->grid.precision == SACX_FP64;
    const int along = dir == 0 ? L.ny : L.nx + 2 * G;
    dim3 g((along + T - 1) / T, NF, 2);
    const DevScalars *none = nullptr;
    if (dir == 0) {
        if (f64) {
            if (pack) hipLaunchKernelGGL(k_pack_x<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, (double *)b0, (double *)b1, 2, none);
            else hipLaunchKernelGGL(k_unpack_x<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, (const double *)b0, (const double *)b1, 2, none);
        } else {
            if (pack) hipLaunchKernelGGL(k_pack_x<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, (float *)b0, (float *)b1, 2, none);
            else hipLaunchKernelGGL(k_unpack_x<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, (const float *)b0, (const float *)b1, 2, none);
        }
    } else {
        if (f64) {
            if (pack) hipLaunchKernelGGL(k_pack_y<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, mx, (double *)b0, (double *)b1, 2, none);
            else hipLaunchKernelGGL(k_unpack_y<double>, g, dim3(T), 0, ctx->stream, fptr<double>(S, NF), NF, L, (const double *)b0, (const double *)b1, 2, none);
        } else {
            if (pack) hipLaunchKernelGGL(k_pack_y<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, mx, (float *)b0, (float *)b1, 2, none);
            else hipLaunchKernelGGL(k_unpack_y<float>, g, dim3(T), 0, ctx->stream, fptr<float>(S, NF), NF, L, (const float *)b0, (const float *)b1, 2, none);
        }
    }
    HIPCHK(hipGetLastError());
    return SACX_OK;
}

// one direction's exchange: every subdomain packs its exchange strips, then
// unpacks the strips its neighbours packed facing it (both sides of the
// direction in one launch where both are exchange sides)
static int domain_exchange(sacx_domain *d, int dir) {
    const int n = d->px * d->py;
    const int lo = 2 * dir, hi = 2 * dir + 1;
    for (int i = 0; i < n; ++i) {
        sacx_ctx *c = (*d->subs)[i];
        void *const *b = (*d->buf)[i].data();
        int rc = SACX_OK;
        if (b[lo] && b[hi]) rc = halo_io_both(c, dir, b[lo], b[hi], true, d->mixed);
        else if (b[lo]) rc = halo_io(c, lo, b[lo], true, d->mixed);
        else if (b[hi]) rc = halo_io(c, hi, b[hi], true, d->mixed);
        if (rc) return rc;
    }
    for (int i = 0; i < n; ++i) {
        sacx_ctx *c = (*d->subs)[i];
        void *const *b = (*d->buf)[i].data();
        // the strip a side receives is the one its neighbour packed facing it
        void *from_lo = b[lo] ? (*d->buf)[(*d->nbr)[i][lo]][hi] : nullptr;
        void *from_hi = b[hi] ? (*d->buf)[(*d->nbr)[i][hi]][lo] : nullptr;
        int rc = SACX_OK;
        if (from_lo && from_hi) rc = halo_io_both(c, dir, from_lo, from_hi, false, d->mixed);
        else if (from_lo) rc = halo_io(c, lo, from_lo, false, d->mixed);
        else if (from_hi) rc = halo_io(c, hi, from_hi, false, d->mixed);
        if (rc) return rc;
    }
    return SACX_OK;
}

int sacx_domain_advance(sacx_domain *d, int32_t nsteps) {
    if (!d) return fail(SACX_EINVAL, "domain must not be NULL");
    if (nsteps < 0) return fail(SACX_EINVAL, "nsteps must be >= 0");
    const int n = d->px * d->py;
    for (int i = 0; i < n; ++i) {
        const sacx_ctx *c = (*d->subs)[i];
        if (c->stage_next) return fail(SACX_ESTATE, "subdomain %d has a step in progress", i);
        for (int side = 0; side < 4; ++side)
            if (c->bc[side] != (*d->bc)[i][side])
                return fail(SACX_ESTATE, "subdomain %d changed its boundaries after the domain was created", i);
        if (c->sur_on) return fail(SACX_ESTATE, "subdomain %d has a learned coefficient", i);
    }
    sacx_ctx *c0 = (*d->subs)[0];
    DeviceGuard dg(c0->device);
    if (!dg.ok) return fail(SACX_EDEVICE, "cannot select the domain's device");
    // One launch per stage (and one for its ghosts) over all subdomains: the
    // subdomains' own launches ran one after the other, each too small for
    // the chip, with 8 pack and unpack launches per stage in a 2 x 2 split.
    // Not where y neighbours have x sides of different kinds (the corners of a
    // subdomain are then what its neighbour has beyond its own sides), not for narrow periodic directions, whose ghosts need fills, not for the
    // one subdomain of a domain with a background, which the list kernels do
    // not read, and not while the stream is captured: a graph must not read
    // tables that a later call may replace.
    bool together = !d->mixed;
    unsigned long long gen = 0;
    for (const sacx_ctx *c : *d->subs) {
        together = together && !c->grid.background_on && !narrow(c, 0) && (c->L.ny == 1 || !narrow(c, 1));
        gen += c->gen;
    }
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (together && nsteps > 0) {
        HIPCHK(hipStreamIsCapturing(c0->stream, &cap));
        if (cap == hipStreamCaptureStatusNone) {
            const bool f64 = c0->grid.precision == SACX_FP64;
            if (!d->built || d->gen_built != gen) {
                const int rc = allocating([&] { return f64 ? domain_build<double>(d, gen) : domain_build<float>(d, gen); });
                if (rc) return rc;
            }
            return f64 ? domain_steps<double>(d, nsteps) : domain_steps<float>(d, nsteps);
        }
    }
    for (int step = 0; step < nsteps; ++step) {
        hipLaunchKernelGGL(k_zero_doubles, dim3(1), dim3(64), 0, c0->stream, d->cmax, 2);
        HIPCHK(hipGetLastError());
        int rc;
        for (int i = 0; i < n; ++i)
            if ((rc = sacx_wave_speeds_max((*d->subs)[i], d->cmax))) return rc;
        for (int s = 0; s < 4; ++s) {
            // without mixed kinds the periodic and open sides need no fill,
            // narrow directions apart
            for (int dir = 0; dir < 2; ++dir) {
                for (int i = 0; i < n; ++i) {
                    sacx_ctx *c = (*d->subs)[i];
                    if ((rc = d->mixed ? sacx_fill_boundaries(c, dir) : fill_narrow(c, stage_input(c), NF, false, dir)))
                        return rc;
                }
                if ((rc = domain_exchange(d, dir))) return rc;
            }
            for (int i = 0; i < n; ++i)
                if ((rc = stage_call((*d->subs)[i], d->cmax, 1, nullptr, d->mixed))) return rc;
        }
    }
    return SACX_OK;
}

}  // extern "C"
