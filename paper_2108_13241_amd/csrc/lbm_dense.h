// Device-side pieces shared by the dense D2Q9 step kernels (one step per launch
// in lbm_kernels.hip, several in lbm_multistep.h): lane moves, the physics
// variants and the kernels' arguments.
#pragma once

#include "lbm_device.h"

namespace lbm {
namespace {

// ------------------------------------------------------------ lane moves --
// DPP move with control word CTRL; a lane whose source lane is outside its row
// or wavefront keeps `edge` (the DPP "old" operand with bound_ctrl off), so the
// end lanes need no select or branch.  Source lanes must be active.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v, uint32_t edge)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v, float edge)
{
    return __builtin_bit_cast(float, dpp_u32<CTRL>(__builtin_bit_cast(uint32_t, v),
                                                   __builtin_bit_cast(uint32_t, edge)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v, double edge)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v), e = __builtin_bit_cast(uint64_t, edge);
    const uint32_t lo = dpp_u32<CTRL>((uint32_t)b, (uint32_t)e);
    const uint32_t hi = dpp_u32<CTRL>((uint32_t)(b >> 32), (uint32_t)(e >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
constexpr int kWaveShr1 = 0x138, kWaveShl1 = 0x130;
// Wave-wide shift by one lane of a full wavefront: UP, lane l receives lane
// l - 1's value (lane 0 keeps edge), else lane l + 1's (lane 63 keeps edge).
template <bool UP, class R>
__device__ __forceinline__ R lane_shift(R v, R edge)
{
    return dpp_move<UP ? kWaveShr1 : kWaveShl1>(v, edge);
}

// Physics variant of a step kernel: plain BGK (no body force, no drag), body
// force, or body force with a drag field; plus kOpen when the lattice has
// open-boundary nodes (lattices without them run kernels free of that branch);
// plus kTRT / kMRT for the two- / multiple-relaxation-time collisions.
enum Phys : int { kBGK = 0, kForced = 1, kDragged = 2, kOpenBC = 4, kTRT = 8, kMRT = 16 };

// Arguments shared by the dense A-B step kernels.
template <class ST>
struct DenseArgs {
    const typename ST::mem *__restrict__ src;
    typename ST::mem *__restrict__ dst;
    const uint8_t *__restrict__ type;
    const uint8_t *__restrict__ nmask;
    const uint32_t *__restrict__ seg_interior;
    const float *__restrict__ alpha;
    const double *__restrict__ bc_val;
    int nx, ny, pitch;
    uint32_t bpr, nblocks;
    typename ST::real omega, gx, gy;
    Rates<typename ST::real> rt;
    int fullway;
};

}  // namespace
}  // namespace lbm
