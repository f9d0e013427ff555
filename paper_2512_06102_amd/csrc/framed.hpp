// framed.hpp -- division of small indices by an env's width: for every 4-cell
// group and observation of the fused RL step, and for the lanes' shares of an env
// in the bit-plane kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace firesim {

// q / d by one fp32 multiply, inv_d = fl(1 / d): the rounding error of
// (q + 1/2) inv_d stays below the 1/(2d) distance of (q + 1/2)/d from an
// integer.  Exact for 0 <= q < 2^14 and 1 <= d <= 2^14 (checked over every
// pair); here q is a dword index (an env has at most 2^16 cells), an
// observation index (side at most 63), a lane or a row count (at most 2^13 rows).
__device__ __forceinline__ int small_div(int q, int d, float inv_d) { return (int)(((float)q + 0.5f) * inv_d); }

}  // namespace firesim
