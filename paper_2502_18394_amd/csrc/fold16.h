// Sums across the lanes of a wave by DPP moves (no LDS round trips).
#pragma once
#include <hip/hip_runtime.h>

namespace spectre {

// Sum over the 16 lanes of a DPP row of 16 values per lane: lane i of a row returns the row's total of value i.
// Reversals of 16, 8, 4 and 2 lanes pair every lane with one that differs in the halving bit, so each step adds the
// half a lane keeps to the half its partner gives away (15 additions instead of 64).
template <int M>
__device__ __forceinline__ float partner16(float v) {
    constexpr int ctrl = (M == 8) ? 0x140 : (M == 4) ? 0x141 : (M == 2) ? 0x1B : 0xB1;   // reverse 16, 8, 4, 2 lanes
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, false));
}
template <int M>
__device__ __forceinline__ void fold16(float (&p)[16], int i) {
    const bool up = i & M;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const float keep = up ? p[j + M] : p[j], give = up ? p[j] : p[j + M];
        p[j] = keep + partner16<M>(give);
    }
}

// Sum of x over the 64 lanes, the same in every lane: four reversals inside the rows of 16, then the four row totals.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double read_lane(double x, int lane) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)u, lane), hi = (unsigned)__builtin_amdgcn_readlane((int)(u >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp_move<0xB1>(x);        // lanes reversed in pairs, fours, eights, sixteens
    x += dpp_move<0x1B>(x);
    x += dpp_move<0x141>(x);
    x += dpp_move<0x140>(x);
    return (read_lane(x, 0) + read_lane(x, 16)) + (read_lane(x, 32) + read_lane(x, 48));
}

}  // namespace spectre
