// sacx_stage_split.hip -- the two-role FP64 stage kernel (k_stage_split), in
// a unit of its own: built, like sacx_stage.hip, without contraction (every
// operation rounds once, in the scheme's order), and with LLVM's iterative
// ILP-maximising scheduler, which measured 2-3 % faster for this kernel and
// 3 % slower for the one-thread tile.
#include "sacx_stage_kernel.h"

namespace sacx {

namespace {

template <int NC, int STAGE>
hipError_t launch_split_s(bool bg, bool sur, dim3 grid, const StageArgs<double> &a, hipStream_t s) {
    if (sur) hipLaunchKernelGGL((k_stage_split<double, NC, STAGE, false, true>), grid, dim3(2 * NC), 0, s, a);
    else if (bg) hipLaunchKernelGGL((k_stage_split<double, NC, STAGE, true>), grid, dim3(2 * NC), 0, s, a);
    else hipLaunchKernelGGL((k_stage_split<double, NC, STAGE, false>), grid, dim3(2 * NC), 0, s, a);
    return hipGetLastError();
}

template <int NC>
hipError_t launch_split_nc(int stage, bool bg, bool sur, dim3 grid, const StageArgs<double> &a, hipStream_t s) {
    switch (stage) {
        case 1: return launch_split_s<NC, 1>(bg, sur, grid, a, s);
        case 2: return launch_split_s<NC, 2>(bg, sur, grid, a, s);
        case 3: return launch_split_s<NC, 3>(bg, sur, grid, a, s);
        default: return launch_split_s<NC, 4>(bg, sur, grid, a, s);
    }
}

template <int NC>
hipError_t split_blocks_nc(bool bg, int *blocks) {
    return bg ? hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_stage_split<double, NC, 1, true>, 2 * NC, 0)
              : hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_stage_split<double, NC, 1, false>, 2 * NC, 0);
}

// one stage's tiles of several subdomains, one block per entry of the list
template <int NC, int STAGE>
__global__ __launch_bounds__(2 * NC, 2) void k_batch_split(const BatchInst<double> *__restrict__ inst,
                                                          const BatchItem *__restrict__ items) {
    __shared__ SplitLds<double, NC, false> lds;
    const BatchItem w = items[listed_tile()];
    const StageArgs<double> a = inst[w.inst].st[STAGE - 1];
    stage_tile_split<double, NC, STAGE, false, false>(a, w.tx, w.ty, lds);
}

template <int NC>
hipError_t launch_batch_split_nc(const BatchArgs<double> &b, int stage, int tiles, hipStream_t s) {
    const dim3 g(tiles), t(2 * NC);
    switch (stage) {
        case 1: hipLaunchKernelGGL((k_batch_split<NC, 1>), g, t, 0, s, b.inst, b.items); break;
        case 2: hipLaunchKernelGGL((k_batch_split<NC, 2>), g, t, 0, s, b.inst, b.items); break;
        case 3: hipLaunchKernelGGL((k_batch_split<NC, 3>), g, t, 0, s, b.inst, b.items); break;
        default: hipLaunchKernelGGL((k_batch_split<NC, 4>), g, t, 0, s, b.inst, b.items); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_batch_split_fp64(const BatchArgs<double> &b, int nc, int stage, int tiles, hipStream_t s) {
    switch (nc) {
        case 64: return launch_batch_split_nc<64>(b, stage, tiles, s);
        case 128: return launch_batch_split_nc<128>(b, stage, tiles, s);
        default: return launch_batch_split_nc<256>(b, stage, tiles, s);
    }
}

hipError_t launch_split_fp64(int stage, int nc, bool bg, bool sur, dim3 grid, const StageArgs<double> &a,
                             hipStream_t s) {
    switch (nc) {
        case 64: return launch_split_nc<64>(stage, bg, sur, grid, a, s);
        case 128: return launch_split_nc<128>(stage, bg, sur, grid, a, s);
        default: return launch_split_nc<256>(stage, bg, sur, grid, a, s);
    }
}

hipError_t split_blocks_per_cu_fp64(int nc, bool bg, int *blocks) {
    switch (nc) {
        case 64: return split_blocks_nc<64>(bg, blocks);
        case 128: return split_blocks_nc<128>(bg, blocks);
        default: return split_blocks_nc<256>(bg, blocks);
    }
}

}  // namespace sacx
