// k_steps for the dense A-B layout, FP64 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_dense_f64(const DevState &s, int cur, int steps)
{
    return steps_placed<F64, kDense>(s, cur, steps);
}

}  // namespace lbm
