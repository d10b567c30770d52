// k_steps for the TILED16 layout, FP64 storage (one file each: they compile in parallel).
#include "lbm_multistep.h"

namespace lbm {

hipError_t launch_steps_tiles_f64(const DevState &s, int cur, int steps)
{
    return steps_placed<F64, kTiles>(s, cur, steps);
}

}  // namespace lbm
