// k_steps for the AA layout after an odd number of steps, FP64 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_aa_f64(const DevState &s, int cur, int steps)
{
    return steps_placed<F64, kDenseOpp>(s, cur, steps);
}

}  // namespace lbm
