#include "star_norm_mma.h"

namespace star {

hipError_t launch_norm_mma_f32(WalkKernelArgs& k, int Wp, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    return launch_mma<RowF32>(k, Wp, num_cu, grid_cap, grid_out, s);
}

}  // namespace star
