// k_steps for the AA layout after an odd number of steps, FP16 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_aa_f16(const DevState &s, int cur, int steps)
{
    return steps_placed<F16S, kDenseOpp>(s, cur, steps);
}

}  // namespace lbm
