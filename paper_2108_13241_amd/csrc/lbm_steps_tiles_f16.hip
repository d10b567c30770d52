// k_steps for the TILED16 layout, FP16 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_tiles_f16(const DevState &s, int cur, int steps)
{
    return steps_placed<F16S, kTiles>(s, cur, steps);
}

}  // namespace lbm
