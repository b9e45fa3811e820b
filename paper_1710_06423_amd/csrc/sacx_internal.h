// sacx_internal.h -- device-side layout, scalar block and kernel launchers
// shared by the HIP translation units of libsacx (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <stdint.h>

#include "sacx.h"

namespace sacx {

// records the calling thread's last-error message and returns `code`
int set_error(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));

#define HIPCHK(expr)                                                                       \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return ::sacx::set_error(SACX_EDEVICE, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                                     __FILE__, __LINE__);                                  \
    } while (0)

constexpr int G = SACX_GHOST;  // ghost cells per side
constexpr int NF = 6;          // evolved fields
constexpr int NBG = 4;         // background fields

// Field storage: one 2-D array per field, (ny + 2G) rows of `pitch` elements.
// Interior element (i, j), i in [-G, nx+G), j in [-G, ny+G), lives at
//   base[xoff + i + (j + G) * pitch]
// xoff is 256 bytes worth of elements so that interior column 0 of every row
// starts on a 256-byte boundary (coalesced, aligned row loads).
struct Layout {
    int nx, ny;
    int pitch;   // elements per row
    int xoff;    // element offset of column 0 within a row
    int rows;    // ny + 2G
    int64_t field_elems;  // elements per field array (rows * pitch, rounded)
};

// Device-resident step scalars.  c accumulators hold the IEEE bit patterns of
// non-negative doubles, so an unsigned 64-bit max is the floating max.
// words over which the blocks of a launch spread their wave-speed maxima
constexpr int kAcc = 8;
struct alignas(128) SpeedWord {
    unsigned long long v[3];   // x, y, z
};

struct DevScalars {
    double t;            // current time
    double dt;           // time step of the step in progress / last taken
    double cmax;         // c_max used by the step in progress
    double t_end;        // end time of the current advance call (<= 0: none)
    // per-step constants derived from dt and c_max (computed once, read by
    // every stage kernel as uniform values)
    double hdt, dt6;     // dt/2, dt/6
    double kx2[4], ky2[4];  // c2 * h_d * c_max per constant class
    double last_cx, last_cy, last_cmax;
    long long steps;     // steps since init
    long long steps0;    // the same when the current advance call began
    int cur;             // slot holding the maxima of the current state
    int active;          // 1 while the step in progress proceeds
    int nonphys;         // sticky: a non-physical state was reduced
    int prev_active;     // `active` of the step before the one in progress, of the same call
    SpeedWord acc[2][kAcc];  // [slot] wave-speed maxima, as the maximum over the words
};

// the maximum over the words of a slot (IEEE bits of non-negative doubles
// order like the doubles)
__host__ __device__ inline unsigned long long speed_max(const SpeedWord (&slot)[kAcc], int d) {
    unsigned long long m = 0ull;
    for (int k = 0; k < kAcc; ++k) {
        const unsigned long long v = slot[k].v[d];
        m = v > m ? v : m;
    }
    return m;
}

// the slot's maxima are cx, cy and cz
__device__ inline void speed_set(SpeedWord (&slot)[kAcc], unsigned long long cx = 0ull, unsigned long long cy = 0ull,
                                 unsigned long long cz = 0ull) {
    for (int k = 0; k < kAcc; ++k) {
        slot[k].v[0] = k ? 0ull : cx;
        slot[k].v[1] = k ? 0ull : cy;
        slot[k].v[2] = k ? 0ull : cz;
    }
}

// Maximum of non-negative values over a full wave, in lane 63.  By register
// lanes (DPP), a few cycles a step; a shuffle goes through the LDS pipe, and
// the eighteen dependent ones of two maxima and a flag were at the end of
// every block.
__device__ __forceinline__ double wave_max(double v) {
    auto step = [](double x, auto ctrl) __attribute__((always_inline)) {
        constexpr int C = decltype(ctrl)::value;
        const int lo = __double2loint(x), hi = __double2hiint(x);
        const int l2 = __builtin_amdgcn_update_dpp(lo, lo, C, 0xf, 0xf, false);
        const int h2 = __builtin_amdgcn_update_dpp(hi, hi, C, 0xf, 0xf, false);
        return fmax(x, __hiloint2double(h2, l2));
    };
    v = step(v, std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8: lane 15 of each row of 16
    v = step(v, std::integral_constant<int, 0x112>{});
    v = step(v, std::integral_constant<int, 0x114>{});
    v = step(v, std::integral_constant<int, 0x118>{});
    v = step(v, std::integral_constant<int, 0x142>{});   // row_bcast 15: lane 31 has rows 0-1, lane 63 rows 2-3
    v = step(v, std::integral_constant<int, 0x143>{});   // row_bcast 31: lane 63 has all
    return v;
}

// the word of this block
__device__ __forceinline__ int acc_word() { return (int)((blockIdx.x + gridDim.x * blockIdx.y) % kAcc); }

// Raise the maxima of a block into a slot.  Atomics on one word are carried
// out one after the other, about 11 ns each: 4096 blocks x 4 waves x 2 maxima
// of an initial state took 380 us at every grid size.  Each block sends one
// maximum per direction, and blocks take turns over kAcc words: the 512 and
// more blocks that end together no longer queue for one word, and no block
// has to read the word first to spare it the atomic.
template <int NW>
__device__ __forceinline__ void raise_speeds(double cx, double cy, int bad, double (&red)[3][NW], DevScalars *sc,
                                             int slot) {
    cx = wave_max(cx);
    cy = wave_max(cy);
    const bool any = __any(bad) != 0;
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) { red[0][w] = cx; red[1][w] = cy; red[2][w] = any ? 1.0 : 0.0; }
    __syncthreads();
    if (threadIdx.x < 3) {
        double m = 0.0;
        for (int k = 0; k < NW; ++k) m = fmax(m, red[threadIdx.x][k]);
        if (threadIdx.x < 2)
            atomicMax(&sc->acc[slot][acc_word()].v[threadIdx.x], (unsigned long long)__double_as_longlong(m));
        else if (m > 0.0)
            atomicOr(&sc->nonphys, 1);
    }
}

// grid constants of the scheme, computed once on the host in FP64
// (reciprocals of grid spacings, closure constants, compression-term scales)
struct SchemeConsts {
    double gamma, gm1, igm1;
    double i12dx, i12dy, idx, idy, i2dx, i2dy;
    double kxs[4], kys[4];   // cshk * h_d * h_d
    double third;
    double gx, gy;           // gravity
    int grav;                // gravity non-zero: its sources are added
};

// constants of the time-step computation
struct StepConsts {
    double cfl, dx, dy;
    double c2[4];
    int ax, ay;  // direction has more than one cell
};

// dt for the step about to start at time t with wave-speed maxima cx, cy: CFL
// time step with the end-time clamp, and the per-step constants derived from it
__device__ inline void step_open(DevScalars *sc, double t_end, const StepConsts &k, double t, int nonphys, double cx,
                                 double cy) {
    sc->t_end = t_end;
    if (nonphys || (t_end > 0.0 && t_end - t <= 1e-12 * t_end)) { sc->active = 0; return; }
    const double dx = k.dx, dy = k.dy;
    double h;
    if (k.ax && k.ay) h = (dx / cx < dy / cy) ? dx / cx : dy / cy;
    else if (k.ax) h = dx / cx;
    else h = dy / cy;
    double dt = k.cfl * h;
    if (t_end > 0.0) dt = (dt < t_end - t) ? dt : t_end - t;
    const double cmax = (k.ax && k.ay) ? (cx > cy ? cx : cy) : (k.ax ? cx : cy);
    sc->dt = dt;
    sc->cmax = cmax;
    sc->last_cx = cx;
    sc->last_cy = cy;
    sc->last_cmax = cmax;
    sc->hdt = 0.5 * dt;
    sc->dt6 = dt / 6.0;
    for (int m = 0; m < 4; ++m) {
        sc->kx2[m] = k.c2[m] * dx * cmax;
        sc->ky2[m] = k.c2[m] * dy * cmax;
    }
    sc->active = 1;
}

// the same by one thread, from the current slot, with the other slot cleared
__device__ inline void step_begin_dev(DevScalars *sc, double t_end, const StepConsts &k) {
    const int cur = sc->cur;
    step_open(sc, t_end, k, sc->t, sc->nonphys, __longlong_as_double((long long)speed_max(sc->acc[cur], 0)),
              __longlong_as_double((long long)speed_max(sc->acc[cur], 1)));
    speed_set(sc->acc[cur ^ 1]);
}

// Both slots' maxima by a wave: lane 32 s + d gets that of slot s, direction d.
// One load per lane instead of a chain of them in one thread.
__device__ __forceinline__ unsigned long long speeds_by_lane(const SpeedWord (&acc)[2][kAcc], int lane) {
    static_assert(kAcc == 8, "a lane per slot, word and direction (of four)");
    unsigned long long v = (lane & 3) < 3 ? acc[lane >> 5][(lane >> 2) & 7].v[lane & 3] : 0ull;
#pragma unroll
    for (int off = 4; off < 32; off <<= 1) {
        const unsigned long long o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    return v;
}
// and clear a slot
__device__ __forceinline__ void speeds_clear_by_lane(SpeedWord (&slot)[kAcc], int lane) {
    if (lane < 32 && (lane & 3) < 3) slot[lane >> 2].v[lane & 3] = 0ull;
}

__device__ inline void step_end_dev(DevScalars *sc) {
    if (!sc->active) return;
    sc->t = sc->t + sc->dt;
    sc->steps = sc->steps + 1;
    sc->cur ^= 1;
}

// Where the cells outside one direction are read: cell i (from -G to n + G - 1)
// is stored at clamp(i, lo, hi), moved by `below` where i < 0 and by `above`
// where i >= n: the periodic image, the edge cell of an open side, or the
// ghost cell itself (exchange sides, periodic directions of fewer than G
// cells, whose ghosts are filled before the stage, and every side in a
// stage-level call, whose ghosts the caller completes).  The stage kernels read
// through this, so that no launch has to fill ghost layers before them: the
// four launches of a fill took 15-19 us per stage at every grid size up to
// 2048^2, where a stage itself takes 25-120 us.
struct SideMap {
    int n, lo, hi, below, above;
    __host__ __device__ __forceinline__ int at(int i) const {
        const int c = i < lo ? lo : (i > hi ? hi : i);
        return c + (i < 0 ? below : 0) + (i >= n ? above : 0);
    }
};

__host__ __device__ inline SideMap side_map(int n, int bc_lo, int bc_hi) {
    SideMap m;
    m.n = n;
    const bool per = bc_lo == SACX_PERIODIC && n >= G;
    m.lo = bc_lo == SACX_OPEN ? 0 : -G;
    m.hi = bc_hi == SACX_OPEN ? n - 1 : n + G - 1;
    m.below = per ? n : 0;
    m.above = per ? -n : 0;
    return m;
}

template <typename real>
struct StageArgs {
    const real *S[NF];    // stage input (differenced; the ghosts of exchange sides filled)
    const real *U[NF];    // step start state (pointwise)
    const real *A[NF];    // RK accumulator (pointwise, stage 4)
    real *out1[NF];       // stage output (w1, w2, w3 or the new state)
    real *out2[NF];       // accumulator output (stage 2)
    const real *BG[NBG];  // static background (optional)
    // elements from one field to the next in every buffer above (the stage
    // kernel addresses field f of a buffer as its field 0 + f * fstride;
    // the host checks that the buffers are laid out that way)
    int64_t fstride;
    Layout L;
    SideMap mx, my;       // where the cells outside are read
    int ty;               // output rows per block
    int nt;               // columns per block (apron included)
    int split;            // FP64 2-D hyper-diffusion tiles without background:
                          // two threads per column (x and y roles)
    SchemeConsts k;
    int hd_cross_on;
    DevScalars *sc;
    // surrogate ratio planes (10: x-face sets then y-face sets, interior
    // cells, periodic): a value >= 0 replaces the plain coefficient ratio of
    // that face, a negative value keeps the plain ratio
    const float *Rs;
    int64_t rs_plane;     // elements per plane
    int rs_pitch;         // elements per row
    // per check tile (row-major, rs_ntx tiles of rs_tile x rs_tile cells per
    // row): 1 where the last check kept the prediction, 0 where it fell back;
    // the planes of a fallen-back tile are not read (its faces take the plain
    // ratio, as its planes' -1 would give)
    const unsigned char *Rk;
    int rs_tile, rs_ntx;
};

// arguments of a tube's step kernel (a whole RK4 step in one launch)
template <typename real>
struct TubeArgs {
    const real *U;       // field 0 of the step's start state (field f at + f * fstride)
    real *out;           // field 0 of the new state
    int64_t fstride;
    Layout L;
    int periodic, open_lo, open_hi;
    SchemeConsts k;
    DevScalars *sc;
    int second;          // this step's U is the step before's out (the pair ends in the state buffer)
};

// arguments of the ratio-field kernels (plain ratios of a state whose halo is
// filled; no background)
template <typename real>
struct RatioArgs {
    const real *S[NF];
    Layout L;
    double gm1, igm1;
};

// device-side surrogate counters.  A check's blocks update one of kStatSlots
// copies of each counter (by block index), so that thousands of blocks do
// not contend for one word; the reader reduces the copies.
constexpr int kStatSlots = 64;
struct HdDevStats {
    unsigned long long tiles_fallback[kStatSlots];
    unsigned long long err_used[kStatSlots];   // IEEE bits of a non-negative double (max)
    unsigned long long err_all[kStatSlots];
    unsigned long long dmax[10];   // per plane max |first difference| of the current check
};

// round to the nearest BF16 value, ties to even (NaN stays a quiet NaN)
__device__ __forceinline__ unsigned short bf16_rne(float f) {
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// ---------------------------------------------------------------- batches
// One instance of a batch: its per-stage kernel arguments, time-step
// constants and ghost-fill description.
template <typename real>
struct BatchInst {
    StageArgs<real> st[4];   // arguments of stages 1..4 (stage inputs, outputs)
    StepConsts sk;
    DevScalars *sc;
    Layout L;
    int periodic_x, periodic_y;
    int oned;                // ny == 1: one-dimensional tiles
    int ntiles;              // tiles of one stage
    int nfill;               // ghost-fill pieces of one stage
    int exchange;            // bit per side (x-, x+, y-, y+): an exchange side
};

// ghost cells (all fields) per ghost-fill piece of a batched instance
constexpr int kBatchFillPiece = 2048;

// an entry of the per-stage work list: one piece (tx) of the ghost fill of an
// instance's stage input (kind BATCH_FILL; piece 0 of a step's first stage
// also takes the step's time step) or one tile of its stage (kind BATCH_TILE)
enum { BATCH_TILE = 0, BATCH_FILL = 1 };
struct BatchItem {
    int inst, tx, ty, kind;
};

// The entry of a stage launch's tile list that a block takes: runs of 4
// neighbouring tiles share an XCD (and the apron in its L2).
__device__ __forceinline__ int listed_tile() {
    const int n = (int)gridDim.x, b = (int)blockIdx.x, i = b / 8;
    return b < n - n % 32 ? ((i / 4) * 8 + b % 8) * 4 + i % 4 : b;
}

// The batch's work is split into one queue per XCD (instances assigned to
// queues by cost); a block serves the queue of the XCD it runs on.
constexpr int kBatchQueues = 8;

// Batch synchronisation words: the abort flag of a dependency wait that
// exceeded its bound (sticky), per queue its work counter (the first of which
// holds the stage launches' non-physical flag) and the count of
// blocks serving it, then per instance the count of completed ghost fills and
// of completed tiles.  All but the abort flag are zeroed before every launch.
enum { BATCH_ABORT = 0, BATCH_QUEUE0 = 1, BATCH_BLOCKS0 = 1 + kBatchQueues, BATCH_SYNC0 = 1 + 2 * kBatchQueues };

template <typename real>
struct BatchArgs {
    const BatchInst<real> *inst;
    int n;
    const BatchItem *items;  // per queue one stage's work list (per instance its fill, then its tiles), queue after queue
    const int *qinst;        // the instances of each queue, queue after queue
    int qoff[kBatchQueues];  // first entry of each queue's list in items
    int qlen[kBatchQueues];  // entries of each queue's list
    int ioff[kBatchQueues + 1];  // prefix offsets of the queues' instances in qinst
    int *sync;               // BATCH_SYNC0 + 2 n words
    int nsteps;
    int spin_limit;          // bound of a dependency wait (polls)
};

// host-side launchers (defined in the .hip units)
template <typename real>
hipError_t launch_stage(int stage, bool hd, bool bg, const StageArgs<real> &a, hipStream_t s);
template <typename real>
hipError_t launch_tube_step(bool hd, int cus, const TubeArgs<real> &a, hipStream_t s);
// stages 1 and 2 (from S = U to out1 and out2 = A) or, `last`, 3 and 4 (from S,
// U and A to out1) of the scheme without hyper-diffusion; no background, no
// exchange sides, at least 8 cells in both directions.  `second`: U is not the
// state buffer but the one that the step before wrote; rows: 8 or 24 per block
template <typename real>
hipError_t launch_pair(bool last, bool second, int rows, const StageArgs<real> &a, hipStream_t s);
// the box kernel, 58 columns x `rows` rows per block (8, or with hyper-diffusion
// 4 in FP64 and 16 in FP32); no background, plain coefficient
template <typename real>
hipError_t launch_box(int stage, bool hd, int rows, const StageArgs<real> &a, hipStream_t s);
template <typename real>
hipError_t stage_blocks_per_cu(int nt, bool hd, bool bg, bool split, int *blocks);
template <typename real>
hipError_t launch_ratio_fields(const RatioArgs<real> &a, float *out, float *d1, int64_t pitch, hipStream_t s);
template <typename real>
hipError_t launch_hd_check(const RatioArgs<real> &a, float *rs, int64_t pitch, double bound, int tile, int metric,
                           HdDevStats *st, unsigned char *kept, hipStream_t s);
struct InputNorm {
    float v[12];   // shift[6], scale[6]
};
template <typename real>
hipError_t launch_cnn_inputs(const RatioArgs<real> &a, const InputNorm &norm, void *x, hipStream_t s);
hipError_t cnn_forward_dev(const void *packed, const void *x, int n, int h, int w, void *a1, void *a2, void *a3,
                           float *out, int64_t oimg, int64_t oplane, int64_t orow, hipStream_t s);
template <typename real>
hipError_t launch_batch(const BatchArgs<real> &b, int nt, int blocks, hipStream_t s);
template <typename real>
hipError_t batch_blocks_per_cu(int nt, int *blocks);
template <typename real>
hipError_t launch_batch_stage(const BatchArgs<real> &b, int nt, int stage, bool hd, int tiles, hipStream_t s);
template <typename real>
hipError_t launch_batch_scalars(const BatchArgs<real> &b, bool prev, bool next, int *nonphys, hipStream_t s);
template <typename real>
hipError_t batch_stage_blocks_per_cu(int nt, bool hd, int *blocks);
// the same with boxes of `rows` rows (launch_box)
template <typename real>
hipError_t launch_batch_box(const BatchArgs<real> &b, int rows, int stage, bool hd, int tiles, hipStream_t s);
// the same with the two-role FP64 tile (2-D instances with hyper-diffusion)
hipError_t launch_batch_split_fp64(const BatchArgs<double> &b, int nc, int stage, int tiles, hipStream_t s);
hipError_t split_blocks_per_cu_fp64(int nc, bool bg, int *blocks);

}  // namespace sacx
