// k_steps for the dense A-B layout, FP32 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_dense_f32(const DevState &s, int cur, int steps)
{
    return steps_placed<F32, kDense>(s, cur, steps);
}

}  // namespace lbm
