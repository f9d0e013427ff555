// bitplane.hpp -- pieces of the kernels that hold an env's state in LDS as
// bit planes (the many-step kernel and the fused RL step): one bit per cell,
// rows of 32-cell words with one zero word between rows and a zero row above
// and below.
#pragma once

#include <cmath>

#include "stepcell.hpp"

namespace firesim {

// Where a front cell's ignition rates come from: the table of the handle
// (static wind), or worked out from the env's or the cells' wind.
enum RateSource { kRatesTable = 0, kRatesEnvWind = 1, kRatesCellWind = 2 };

// Orders one wave's LDS writes before its later LDS reads by other lanes of
// the same wave.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Bits of a 32-cell word at column 32 w that lie in columns [lo, hi).
__device__ __forceinline__ uint32_t column_mask(int w, int lo, int hi)
{
    const int a = min(max(lo - 32 * w, 0), 32), b = min(max(hi - 32 * w, 0), 32);
    const uint32_t below_b = b >= 32 ? ~0u : (1u << b) - 1u;
    const uint32_t below_a = a >= 32 ? ~0u : (1u << a) - 1u;
    return below_b & ~below_a;
}

// Four flag bits spread to the low bit of four bytes.
__device__ __forceinline__ uint32_t spread4(uint32_t x) { return ((x & 0xFu) * 0x00204081u) & 0x01010101u; }

// phi of the eight edges into a cell, summed over the burning sources in ascending
// direction order (win: 3 x 3 burning window, rows up / middle / down of 3
// bits).  Adding 0 for a source that does not burn leaves the sum as it is.
__device__ __forceinline__ float rate_sum(const float4& a, const float4& b, uint32_t win)
{
    auto on = [&](float x, int bit) {
        return __int_as_float(__float_as_int(x) & __builtin_amdgcn_sbfe((int)win, bit, 1));
    };
    float l = 0.0f;
    l = l + on(a.x, 3);
    l = l + on(a.y, 6);
    l = l + on(a.z, 7);
    l = l + on(a.w, 8);
    l = l + on(b.x, 5);
    l = l + on(b.y, 2);
    l = l + on(b.z, 1);
    l = l + on(b.w, 0);
    return l;
}

// A burning cell with 24-bit draw k stays when k 2^-24 < p, i.e. k < ceil(2^24 p).
inline uint32_t keep_threshold(float p)
{
    if (!(p > 0.0f)) return 0u;
    if (p >= 1.0f) return 1u << 24;
    return (uint32_t)std::ceil((double)p * 16777216.0);
}

}  // namespace firesim
