// sacx_box.hip -- the box stage kernel, the two-stage kernel and the tube's step kernel, double arithmetic.
#include "sacx_box_kernel.h"
#include "sacx_tile_pair.h"
#include "sacx_tube.h"

namespace sacx {

template hipError_t launch_box<double>(int, bool, int, const StageArgs<double> &, hipStream_t);
template hipError_t launch_batch_box<double>(const BatchArgs<double> &, int, int, bool, int, hipStream_t);
template hipError_t launch_pair<double>(bool, bool, int, const StageArgs<double> &, hipStream_t);
template hipError_t launch_tube_step<double>(bool, int, const TubeArgs<double> &, hipStream_t);

}  // namespace sacx
