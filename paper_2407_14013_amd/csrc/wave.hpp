// Cross-lane helpers of a 64-wide wave (gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace wc {

// v from the lane that the DPP control names (a permutation within a row of 16 lanes)
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(x >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// Sum over the 16 lanes of each row of lanes, delivered to all of them.  DPP
// moves stay in the vector pipeline; a shuffle is a round trip through the LDS
// crossbar (an FP64 one two of them), and these sums sit on latency chains.
__device__ __forceinline__ double row16_sum(double v) {
    v += dpp_mov<0xB1>(v);   // lane ^ 1
    v += dpp_mov<0x4E>(v);   // lane ^ 2
    v += dpp_mov<0x141>(v);  // the other quad of the eight (row_half_mirror)
    v += dpp_mov<0x140>(v);  // the other eight of the row (row_mirror)
    return v;
}

// Sum over the four lanes that share a place in their rows (l, l + 16, l + 32,
// l + 48), delivered to all four, by the lane-swap instructions.
__device__ __forceinline__ double rows4_sum(double v) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    auto pair = [](unsigned a0, unsigned a1) {
        return __longlong_as_double((static_cast<long long>(a1) << 32) | static_cast<long long>(a0));
    };
    long long x = __double_as_longlong(v);
    unsigned lo = static_cast<unsigned>(x), hi = static_cast<unsigned>(x >> 32);
    u2 l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    u2 h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = pair(l.x, h.x) + pair(l.y, h.y);
    x = __double_as_longlong(v);
    lo = static_cast<unsigned>(x);
    hi = static_cast<unsigned>(x >> 32);
    l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return pair(l.x, h.x) + pair(l.y, h.y);
}

// Sum over the whole wave, delivered to every lane.
__device__ __forceinline__ double wave_sum_all(double v) { return rows4_sum(row16_sum(v)); }

}  // namespace wc
