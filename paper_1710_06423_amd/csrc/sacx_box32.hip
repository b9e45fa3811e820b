// sacx_box32.hip -- the box stage kernel, the two-stage kernel and the tube's step kernel, float arithmetic.
#include "sacx_box_kernel.h"
#include "sacx_tile_pair.h"
#include "sacx_tube.h"

namespace sacx {

template hipError_t launch_box<float>(int, bool, int, const StageArgs<float> &, hipStream_t);
template hipError_t launch_batch_box<float>(const BatchArgs<float> &, int, int, bool, int, hipStream_t);
template hipError_t launch_pair<float>(bool, bool, int, const StageArgs<float> &, hipStream_t);
template hipError_t launch_tube_step<float>(bool, int, const TubeArgs<float> &, hipStream_t);

}  // namespace sacx
