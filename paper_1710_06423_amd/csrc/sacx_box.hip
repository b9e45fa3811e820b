// sacx_box.hip -- the box stage kernel, double arithmetic.
#include "sacx_box_kernel.h"

namespace sacx {

template hipError_t launch_box<double>(int, bool, int, const StageArgs<double> &, hipStream_t);
template hipError_t launch_batch_box<double>(const BatchArgs<double> &, int, int, bool, int, hipStream_t);

}  // namespace sacx
