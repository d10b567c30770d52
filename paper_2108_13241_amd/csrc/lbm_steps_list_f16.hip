// k_steps for the INDIRECT layout, FP16 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_list_f16(const DevState &s, int cur, int steps)
{
    return steps_placed<F16S, kList>(s, cur, steps);
}

}  // namespace lbm
