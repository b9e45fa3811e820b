// sacx_batch.hip -- FP64 instantiation of the batched launches (built without
// contraction, like the FP64 stage kernel).
#include "sacx_batch_kernel.h"

namespace sacx {

template hipError_t launch_batch<double>(const BatchArgs<double> &, int, int, hipStream_t);
template hipError_t batch_blocks_per_cu<double>(int, int *);
template hipError_t launch_batch_stage<double>(const BatchArgs<double> &, int, int, bool, int, hipStream_t);
template hipError_t launch_batch_scalars<double>(const BatchArgs<double> &, bool, bool, int *, hipStream_t);
template hipError_t batch_stage_blocks_per_cu<double>(int, bool, int *);

}  // namespace sacx
