// Reductions and scans over the 64 lanes of a wave through DPP row shifts and
// row broadcasts (no LDS traffic).  Every lane of the wave must be active.
#pragma once
#include "kernels.hpp"

namespace emppi {

// DPP controls: shift right by n within a row of 16 lanes, and the broadcast
// of a row's last lane to the next row(s).
constexpr int DPP_SHR1 = 0x111, DPP_SHR2 = 0x112, DPP_SHR4 = 0x114, DPP_SHR8 = 0x118;
constexpr int DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143;

// v of the lane the control names, `old` where it names none (or the row is
// not in the mask).
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int dpp_or(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ float dpp_or(float old, float v) {
    return __int_as_float(dpp_or<CTRL, ROWS>(__float_as_int(old), __float_as_int(v)));
}

// Unsigned minimum over the wave, the same in every lane.  The neutral
// element as the value of absent lanes lets each step be one instruction.
__device__ __forceinline__ unsigned wave_umin(unsigned u) {
    auto step = [](unsigned a, int b) { return min(a, static_cast<unsigned>(b)); };
    const int none = -1;
    u = step(u, dpp_or<DPP_SHR1>(none, static_cast<int>(u)));
    u = step(u, dpp_or<DPP_SHR2>(none, static_cast<int>(u)));
    u = step(u, dpp_or<DPP_SHR4>(none, static_cast<int>(u)));
    u = step(u, dpp_or<DPP_SHR8>(none, static_cast<int>(u)));
    u = step(u, dpp_or<DPP_BCAST15>(none, static_cast<int>(u)));
    u = step(u, dpp_or<DPP_BCAST31>(none, static_cast<int>(u)));
    return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(u), WAVE - 1));
}

// Minimum over the wave, the same in every lane, through the floats' ordered
// keys (a positive NaN never is the minimum).
__device__ __forceinline__ float wave_min(float v) { return dkey_value(wave_umin(dkey(v))); }

// Inclusive sums over the wave.
__device__ __forceinline__ int wave_scan(int v) {
    v += dpp_or<DPP_SHR1>(0, v);
    v += dpp_or<DPP_SHR2>(0, v);
    v += dpp_or<DPP_SHR4>(0, v);
    v += dpp_or<DPP_SHR8>(0, v);
    v += dpp_or<DPP_BCAST15, 0xA>(0, v);
    v += dpp_or<DPP_BCAST31, 0xC>(0, v);
    return v;
}
__device__ __forceinline__ int wave_sum(int v) {
    return __builtin_amdgcn_readlane(wave_scan(v), WAVE - 1);
}

}  // namespace emppi
