// Device helpers shared by the solver and network kernels (wave64, gfx950).
#pragma once

#include <math.h>

#include "pa_internal.h"

namespace pa {

__device__ __forceinline__ double wave_sum(double v) {
    // Butterfly over the 64 lanes; the fixed pattern makes the result order-deterministic.
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sums over four elements of the Eq. (4) absolute and the Eq. (2) squared differences.
__device__ __forceinline__ double abs_dev(float4 a, float4 b) {
    return (fabs((double)a.x - (double)b.x) + fabs((double)a.y - (double)b.y)) +
           (fabs((double)a.z - (double)b.z) + fabs((double)a.w - (double)b.w));
}

__device__ __forceinline__ double sq_dev(float4 a, float4 b) {
    const double dx = (double)a.x - (double)b.x, dy = (double)a.y - (double)b.y;
    const double dz = (double)a.z - (double)b.z, dw = (double)a.w - (double)b.w;
    return (dx * dx + dy * dy) + (dz * dz + dw * dw);
}

__device__ __forceinline__ unsigned long long lanemask_lt() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

}  // namespace pa
