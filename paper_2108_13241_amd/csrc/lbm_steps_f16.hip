// k_steps for FP16 storage (one file per storage type: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_f16(const DevState &s, int cur, int steps)
{
    return steps_typed<F16S>(s, cur, steps);
}

}  // namespace lbm
