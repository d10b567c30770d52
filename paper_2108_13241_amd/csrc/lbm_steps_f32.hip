// k_steps for FP32 storage (one file per storage type: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_f32(const DevState &s, int cur, int steps)
{
    return steps_typed<F32>(s, cur, steps);
}

}  // namespace lbm
