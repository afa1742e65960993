// Values of a wave's lanes moved and added up within vector instructions, and over the waves of a workgroup.  Included by .hip files
// only; everything has internal linkage and is called by the whole wave.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace tns {
namespace {

constexpr int kWave = 64;

// Moves inside a row of sixteen lanes are part of a vector instruction (DPP); a shuffle is a round trip through the LDS unit, some
// sixty cycles each, and what waits for a shuffle waits for all of it.  Called by the whole wave.
template <int LANE>
__device__ __forceinline__ int32_t row_read(int32_t v) { return __builtin_amdgcn_update_dpp(0, v, 0x150 + LANE, 0xf, 0xf, true); }      // of lane LANE of the row
template <int BY>
__device__ __forceinline__ int32_t row_up(int32_t v) { return __builtin_amdgcn_update_dpp(0, v, 0x110 + BY, 0xf, 0xf, true); }          // of the lane BY below, 0 at the row's begin

__device__ __forceinline__ int32_t row_inclusive_scan(int32_t v) {
    v += row_up<1>(v);
    v += row_up<2>(v);
    v += row_up<4>(v);
    return v + row_up<8>(v);
}
__device__ __forceinline__ int32_t wave_inclusive_scan(int32_t v) {
    v = row_inclusive_scan(v);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);            // rows 1 and 3: what the row before them has in its last lane
    return v + __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);      // rows 2 and 3: what lane 31 has
}
// Sum over the first n of the workgroup's waves (at most sixteen), whose own sums lie in LDS: a value per lane and one LDS access, where
// a loop over the waves waits for one access after the other.
__device__ __forceinline__ int32_t sum_of_waves(const int32_t* s_wave_sum, int n, int lane) {
    const int w = lane & 15, v = s_wave_sum[w];
    return __builtin_amdgcn_readlane(row_inclusive_scan(w < n ? v : 0), 15);
}
__device__ __forceinline__ int32_t wave_sum(int32_t v) { return __builtin_amdgcn_readlane(wave_inclusive_scan(v), kWave - 1); }

// The same for 64-bit values.
template <int CTRL, int ROWS, bool ZERO>
__device__ __forceinline__ int64_t lanes_moved64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, ZERO);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)v >> 32), CTRL, ROWS, 0xf, ZERO);
    return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ int64_t row_inclusive_scan64(int64_t v) {
    v += lanes_moved64<0x111, 0xf, true>(v);
    v += lanes_moved64<0x112, 0xf, true>(v);
    v += lanes_moved64<0x114, 0xf, true>(v);
    return v + lanes_moved64<0x118, 0xf, true>(v);
}
__device__ __forceinline__ int64_t wave_inclusive_scan64(int64_t v) {
    v = row_inclusive_scan64(v);
    v += lanes_moved64<0x142, 0xa, false>(v);
    return v + lanes_moved64<0x143, 0xc, false>(v);
}
__device__ __forceinline__ int64_t read_lane64(int64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ int64_t wave_sum64(int64_t v) { return read_lane64(wave_inclusive_scan64(v), kWave - 1); }
__device__ __forceinline__ int64_t sum_of_waves64(const int64_t* s_wave_sum, int n, int lane) {
    const int w = lane & 15;
    const int64_t v = s_wave_sum[w];
    return read_lane64(row_inclusive_scan64(w < n ? v : 0), 15);
}

}  // namespace
}  // namespace tns
