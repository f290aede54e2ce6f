// Count task, f32, tile kernels (see mmlike_tile_impl.h)
#include "mmlike_tile_impl.h"

namespace amulet {
template hipError_t launch_mmlike_tile<float, TASK_COUNT_GT>(int, int, const TilePlan &, const TileArgs<float> &, hipStream_t);
}
