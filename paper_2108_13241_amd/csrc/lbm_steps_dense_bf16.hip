// k_steps for the dense A-B layout, BF16 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_dense_bf16(const DevState &s, int cur, int steps)
{
    return steps_placed<BF16S, kDense>(s, cur, steps);
}

}  // namespace lbm
