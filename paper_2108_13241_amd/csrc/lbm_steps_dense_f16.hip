// k_steps for the dense A-B layout, FP16 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_dense_f16(const DevState &s, int cur, int steps)
{
    return steps_placed<F16S, kDense>(s, cur, steps);
}

}  // namespace lbm
