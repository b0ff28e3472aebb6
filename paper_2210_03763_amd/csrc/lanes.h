// Exchanges and sums over the lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>

namespace ttn {

// Lane exchanges inside a row of 16 lanes without a trip through LDS (DPP): the
// value of the lane the control word names, 0 where that lane does not exist
// or the row is masked off.
template <int CTRL, int ROWS = 0xf>
__device__ inline double dpp_move(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffff), CTRL, ROWS, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int DPP_QUAD_XOR1 = 0xB1, DPP_QUAD_XOR2 = 0x4E, DPP_ROW_SHL1 = 0x101, DPP_ROW_SHR1 = 0x111,
              DPP_ROW_SHR2 = 0x112, DPP_ROW_SHR4 = 0x114, DPP_ROW_SHR8 = 0x118, DPP_ROW_MIRROR = 0x140, DPP_ROW_HALF_MIRROR = 0x141,
              DPP_ROW_BCAST15 = 0x142, DPP_ROW_BCAST31 = 0x143;

__device__ inline double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), lane);
    const unsigned hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// sum over each row of 16 lanes, in all of its lanes
__device__ inline double row_total(double v) {
    v += dpp_move<DPP_QUAD_XOR1>(v);
    v += dpp_move<DPP_QUAD_XOR2>(v);
    v += dpp_move<DPP_ROW_HALF_MIRROR>(v);
    return v + dpp_move<DPP_ROW_MIRROR>(v);
}

// sum over a whole wave (all 64 lanes active), the same value in every lane
__device__ inline double wave_total(double v) {
    v += dpp_move<DPP_ROW_SHR1>(v);
    v += dpp_move<DPP_ROW_SHR2>(v);
    v += dpp_move<DPP_ROW_SHR4>(v);
    v += dpp_move<DPP_ROW_SHR8>(v);
    v += dpp_move<DPP_ROW_BCAST15, 0xa>(v);
    v += dpp_move<DPP_ROW_BCAST31, 0xc>(v);
    return lane_value(v, 63);
}

}  // namespace ttn
