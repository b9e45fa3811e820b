// sacx_batch32.hip -- FP32 instantiation of the batched launches (built with
// multiply-add contraction, like the FP32 stage kernel).
#include "sacx_batch_kernel.h"

namespace sacx {

template hipError_t launch_batch<float>(const BatchArgs<float> &, int, int, hipStream_t);
template hipError_t batch_blocks_per_cu<float>(int, int *);
template hipError_t launch_batch_stage<float>(const BatchArgs<float> &, int, int, bool, int, hipStream_t);
template hipError_t launch_batch_scalars<float>(const BatchArgs<float> &, bool, bool, int *, hipStream_t);
template hipError_t batch_stage_blocks_per_cu<float>(int, bool, int *);

}  // namespace sacx
