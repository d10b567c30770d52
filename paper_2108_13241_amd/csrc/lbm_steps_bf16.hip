// k_steps for BF16 storage (one file per storage type: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_bf16(const DevState &s, int cur, int steps)
{
    return steps_typed<BF16S>(s, cur, steps);
}

}  // namespace lbm
