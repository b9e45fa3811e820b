// sacx_box_kernel.h -- the box stage kernel and its launchers, as templates; each
// precision is instantiated in a unit of its own with the contraction rule of
// that precision's stage kernel.
#pragma once

#include "sacx_stage_kernel.h"
#include "sacx_tile_box.h"

namespace sacx {

template <typename real, int W, int R, int STAGE, bool HD>
__global__ __launch_bounds__(64 * W, R == 1 ? 4 : 2) void k_stage_box(StageArgs<real> a) {
    __shared__ BoxLds<real, W, R, HD> lds;
    int tx, ty;
    xcd_tile<4>(tx, ty);
    stage_tile_box<real, W, R, STAGE, HD>(a, tx, ty, lds);
}

template <typename real, int W, int R, bool HD>
static hipError_t launch_box_r(int stage, const StageArgs<real> &a, hipStream_t s) {
    const dim3 g((a.L.nx + 57) / 58, (a.L.ny + W * R - 1) / (W * R)), t(64 * W);
    switch (stage) {
        case 1: hipLaunchKernelGGL((k_stage_box<real, W, R, 1, HD>), g, t, 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_stage_box<real, W, R, 2, HD>), g, t, 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_stage_box<real, W, R, 3, HD>), g, t, 0, s, a); break;
        default: hipLaunchKernelGGL((k_stage_box<real, W, R, 4, HD>), g, t, 0, s, a); break;
    }
    return hipGetLastError();
}

// one stage's blocks of several subdomains: boxes of 58 columns x R rows per
// wave, and of tubes 506 cells
template <typename real, int W, int R, int STAGE, bool HD>
__global__ __launch_bounds__(64 * W, R == 1 ? 4 : 2) void k_batch_box(const BatchInst<real> *__restrict__ inst,
                                                                     const BatchItem *__restrict__ items) {
    __shared__ union {
        BoxLds<real, W, R, HD> box;
        TubeLds<real, 64 * W> tube;
    } lds;
    const BatchItem w = items[listed_tile()];
    const StageArgs<real> a = inst[w.inst].st[STAGE - 1];
    if (inst[w.inst].oned) stage_tile_1d<real, 64 * W, STAGE, HD>(a, w.tx, lds.tube);
    else stage_tile_box<real, W, R, STAGE, HD>(a, w.tx, w.ty, lds.box);
}

template <typename real, int W, int R, bool HD>
static hipError_t launch_batch_box_r(const BatchArgs<real> &b, int stage, int tiles, hipStream_t s) {
    const dim3 g(tiles), t(64 * W);
    switch (stage) {
        case 1: hipLaunchKernelGGL((k_batch_box<real, W, R, 1, HD>), g, t, 0, s, b.inst, b.items); break;
        case 2: hipLaunchKernelGGL((k_batch_box<real, W, R, 2, HD>), g, t, 0, s, b.inst, b.items); break;
        case 3: hipLaunchKernelGGL((k_batch_box<real, W, R, 3, HD>), g, t, 0, s, b.inst, b.items); break;
        default: hipLaunchKernelGGL((k_batch_box<real, W, R, 4, HD>), g, t, 0, s, b.inst, b.items); break;
    }
    return hipGetLastError();
}

template <typename real>
hipError_t launch_batch_box(const BatchArgs<real> &b, int rows, int stage, bool hd, int tiles, hipStream_t s) {
    if constexpr (sizeof(real) == 4) {
        if (hd && rows == 16) return launch_batch_box_r<real, 8, 2, true>(b, stage, tiles, s);
    }
    return hd ? launch_batch_box_r<real, 8, 1, true>(b, stage, tiles, s)
              : launch_batch_box_r<real, 8, 1, false>(b, stage, tiles, s);
}

// rows: 8 (one row per wave) or, with hyper-diffusion, 4 in FP64 (four waves)
// and 16 in FP32 (two rows per wave)
template <typename real>
hipError_t launch_box(int stage, bool hd, int rows, const StageArgs<real> &a, hipStream_t s) {
    if constexpr (sizeof(real) == 4) {
        if (hd && rows == 16) return launch_box_r<real, 8, 2, true>(stage, a, s);
    } else {
        if (hd && rows == 4) return launch_box_r<real, 4, 1, true>(stage, a, s);
    }
    return hd ? launch_box_r<real, 8, 1, true>(stage, a, s) : launch_box_r<real, 8, 1, false>(stage, a, s);
}

}  // namespace sacx
