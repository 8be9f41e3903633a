// wave_scan.h -- inclusive scan over a wavefront in vector-ALU lane moves (no
// LDS round trips): four shifts inside each row of 16 lanes, then the last lane
// of a row into the next row and the last lane of the lower half into the
// upper.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tsattn {

// The value that lane move CTRL brings into this lane, zero where it brings
// none (rows outside kRows, or no source lane).
template <int CTRL, int kRows>
__device__ __forceinline__ int lane_move(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, kRows, 0xf, false);
}
template <int CTRL, int kRows>
__device__ __forceinline__ uint64_t lane_move(uint64_t x) {
    const uint32_t lo = (uint32_t)lane_move<CTRL, kRows>((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)lane_move<CTRL, kRows>((int)(uint32_t)(x >> 32));
    return (uint64_t)hi << 32 | lo;
}
template <int CTRL, int kRows>
__device__ __forceinline__ double lane_move(double x) {
    return __longlong_as_double((long long)lane_move<CTRL, kRows>((uint64_t)__double_as_longlong(x)));
}

// add(x, zero) must be x.  Other types bring their own lane_move.
template <typename T, typename Add>
__device__ __forceinline__ T wave_incl_scan(T x, Add add) {
    constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    x = add(x, lane_move<kRowShr + 1, 0xf>(x));
    x = add(x, lane_move<kRowShr + 2, 0xf>(x));
    x = add(x, lane_move<kRowShr + 4, 0xf>(x));
    x = add(x, lane_move<kRowShr + 8, 0xf>(x));
    x = add(x, lane_move<kRowBcast15, 0xa>(x));
    return add(x, lane_move<kRowBcast31, 0xc>(x));
}
template <typename T>
__device__ __forceinline__ T wave_incl_scan(T x) {
    return wave_incl_scan(x, [](T a, T b) { return a + b; });
}

}  // namespace tsattn
