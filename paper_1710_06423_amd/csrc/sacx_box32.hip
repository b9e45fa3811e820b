// sacx_box32.hip -- the box stage kernel, float arithmetic.
#include "sacx_box_kernel.h"

namespace sacx {

template hipError_t launch_box<float>(int, bool, int, const StageArgs<float> &, hipStream_t);
template hipError_t launch_batch_box<float>(const BatchArgs<float> &, int, int, bool, int, hipStream_t);

}  // namespace sacx
